// Golden-label pipeline (Sec. 2.2, Eqs. 7-11) over raw indexer logits
// S[i][l][s] of one window: for every decoding step i and layer l the
// softmax over the entries s (Eq. 7) and its top-p set (Eq. 8: the smallest
// set of the most probable entries whose mass reaches p, more probable first,
// lower index first among equals), the votes of the L layers per entry
// (Eq. 9), the golden set of entries with at least theta votes (Eq. 10), and
// the union of the golden sets over the window (Eq. 11).
//
// The top-p decision is exact: a weight is exp(S - max S) evaluated by one
// fixed float32 method (Cody-Waite reduction with the fdlibm split of ln 2,
// Taylor series of degree 7 in Horner form with fused multiply-adds), held as
// the integer q = floor(w * 2^40); masses are integer sums, so their order
// does not matter, and a set reaches p = num / den when
// (its mass) * den >= num * Z in 128-bit integers.
//
// golden_scan_kernel -- rows of more than 16,384 entries: one 512-thread
//   workgroup per slice of at most 16,384 entries, which is read once into
//   registers.  It leaves the slice's largest entries (every entry with a key
//   at or above the slice's threshold, about 130 of 16,384), its maximum and
//   the sum of the approximate weights of all other entries in the row's own
//   bitmap words, which the next kernels overwrite.
// golden_row_kernel -- one 256-thread workgroup per scanned row takes in the
//   listed entries.  Their masses are exact; the mass of all other entries lies
//   in an interval that bounds every rounding of the approximate sum.  A
//   1024-bin LDS histogram of the listed masses finds the bin where the
//   cumulative mass reaches p (once more inside a bin of many entries), whose
//   entries are ranked directly: the threshold key T and the number of entries
//   equal to T that the set needs.  When both ends of the interval give the
//   same answer it is the exact one, and the row's bitmap is assembled in LDS.
// golden_exact_kernel -- one 512-thread workgroup per row that is not scanned,
//   which is read once into registers, or that the row kernel left open (a flat
//   row, whose set reaches below the listed entries, or a boundary inside the
//   interval), which is read twice more: a 4096-bin LDS histogram of the exact
//   masses by the top 12 bits of each logit's order key, whose descending scan
//   finds the bin where the cumulative mass reaches p, then the bitmap of the
//   bins above it (wavefront ballots) with the entries of that bin staged in
//   LDS (or refined by passes over the row when they do not fit).  Up to 64 of
//   them are compared with one another, more take two 10-bit digit rounds.
// golden_vote_kernel -- one thread per (sequence, one or two steps, bitmap
//   word): the votes of the L layers for 32 entries as bit-sliced counters, the
//   theta test, an OR into the label bitmap and the golden-set sizes.
// golden_compact_kernel -- one workgroup per sequence: label bitmap to
//   ascending entry ids.
//
// What a window takes depends on its logits, as only rows whose set lies within
// the listed entries are settled by the scan.  64 steps, 21 layers, 131,072
// entries (705 MB), us, against reading every row three times: 1 entry in 256 far
// above the others 452 -> 165 (scan 120, rows 27, exact 4.5 with no row left to it,
// votes 9, labels 5); the second half masked 399 -> 163; one row of those open
// (about one window in ten) about 90 more, as one workgroup then reads it alone;
// standard normal logits, every row open, 1,450 to 1,850 -> 510 to 920 from process
// to process; p = 0.9 of the peaked rows 451 -> 220, p = 1, every row open, 512 -> 443.
#include "golden_geometry.h"
#include "lsa_internal.h"

namespace lsa {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kBins = 4096;     // first digit: top 12 bits of the order key
constexpr int kSubBins = 1024;  // two more digits of 10 bits
constexpr int kBinsPerThread = kBins / kThreads;
constexpr int kSubPerThread = kSubBins / kThreads;
constexpr int kCand = 3072;     // entries of the threshold bin staged in LDS
constexpr int kFewCand = 64;    // entries that are compared with one another instead
constexpr int kScanVec = kGoldenSliceVecs / kThreads;  // float4s of a slice a thread holds
static_assert(kThreads == kGoldenScanThreads, "scan geometry");

struct u128 {
  uint64_t hi, lo;
};

__device__ __forceinline__ u128 mul64(uint64_t a, uint64_t b) { return {__umul64hi(a, b), a * b}; }
__device__ __forceinline__ bool ge128(u128 a, u128 b) { return a.hi > b.hi || (a.hi == b.hi && a.lo >= b.lo); }

// Weight of logit s in units of 2^-40 of the largest weight (that of m):
// floor(w * 2^40) with w = exp(s - m) by the fixed float32 method described
// above, which is 0 below -64 (as is the floor from -27.8 on, so that x may be
// held at -64).  w * 2^24 is a float32 and its floor, at most 2^24, an integer
// float32; the difference is exact, and its first 16 bits are the rest of the
// floor.  Branch-free: 25 instructions, where taking the floor from w's bits by
// variable 64-bit shifts took about 60 (1,344 rows of 16,384: 66 -> 58 us a call).
__device__ __forceinline__ uint64_t mass_of(float s, float m) {
  const float log2e = 1.44269502e+00f;
  const float ln2_hi = 6.9314575195e-01f;
  const float ln2_lo = 1.4286067653e-06f;
  const float x = fmaxf(__fsub_rn(s, m), -64.0f);
  const float k = __builtin_rintf(x * log2e);
  float r = __builtin_fmaf(-k, ln2_hi, x);
  r = __builtin_fmaf(-k, ln2_lo, r);
  float p = 1.0f / 5040.0f;
  p = __builtin_fmaf(p, r, 1.0f / 720.0f);
  p = __builtin_fmaf(p, r, 1.0f / 120.0f);
  p = __builtin_fmaf(p, r, 1.0f / 24.0f);
  p = __builtin_fmaf(p, r, 1.0f / 6.0f);
  p = __builtin_fmaf(p, r, 1.0f / 2.0f);
  p = __builtin_fmaf(p, r, 1.0f);
  p = __builtin_fmaf(p, r, 1.0f);
  const float t = __builtin_amdgcn_ldexpf(p, (int)k + 24);  // w * 2^24
  const uint32_t hi = (uint32_t)t;
  const uint32_t lo = (uint32_t)(__fsub_rn(t, (float)hi) * 65536.0f);
  return ((uint64_t)hi << 16) | lo;
}

__device__ __forceinline__ uint32_t key_of(float f) { return order_key<kKeysFromF32>(__float_as_uint(f)); }

__device__ __forceinline__ float logit_of(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

// (The lane number is opaque: the six addresses would otherwise stay in
// registers from one reduction to the next.)
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "one or two words");
  typedef int words __attribute__((ext_vector_type(sizeof(T) / 4)));
  int at = 4 * ((int)threadIdx.x & 63);
  asm volatile("" : "+v"(at));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    words w = __builtin_bit_cast(words, v);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = __builtin_amdgcn_ds_bpermute(at ^ (4 * off), w[i]);
    v = op(v, __builtin_bit_cast(T, w));
  }
  return v;
}

// Exclusive prefix sum over the workgroup in thread order; *total gets the sum.
__device__ __forceinline__ uint64_t block_scan_u64(uint64_t v, uint64_t* wave_tot, uint64_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint64_t x = wave_tot[w];
    before += w < wave ? x : 0ull;
    all += x;
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float fmin2(float a, float b) { return a < b ? a : b; }
__device__ __forceinline__ float fmax2(float a, float b) { return a > b ? a : b; }

// The value of lane i ^ 1, of lane i ^ 2, and (once four, eight adjacent lanes
// agree) of the other four of eight and the other eight of sixteen lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

// op of this lane's value and that of lane ^ 16
template <class Op>
__device__ __forceinline__ float with16(float x, Op op) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(s[0]), __uint_as_float(s[1]));
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// A workgroup barrier for data in LDS only (a fenced one also waits for memory).
__device__ __forceinline__ void lds_barrier() {
  constexpr int kWaitLds = 0xF | (0x3 << 14) | (0x7 << 4);  // s_waitcnt lgkmcnt(0)
  __asm__ volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(kWaitLds);
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

// Bound: one read of the logits (HBM), against about ten vector instructions
// per entry (an exponential among them).  The slice stays in registers, so the
// maximum, the threshold and the sum need no second read; four workgroups per
// CU overlap one's loads with another's arithmetic.  705 MB in 120 us, 5.9
// TB/s; without the listing 114 us.  (Listing straight to memory took 138 us,
// one wavefront per 4,096 entries with no barriers 208 us, and a persistent
// grid that prefetches the next slice 169 us.)  The threshold is the
// smallest of 32 group maxima (512 entries each), which about 130 entries of
// 16,384 reach whatever their distribution; where those do not fit the list
// (short slices, many equal logits) 16, 8, 4 or 2 groups raise it, and past
// those nothing is listed and the threshold lies above the slice's maximum.
__global__ void __launch_bounds__(kThreads, 8)
golden_scan_kernel(GoldenTable gt, GoldenArgs a, int64_t first_slice) {
  __shared__ float list_x[kWaves][kSliceListMax];
  __shared__ uint16_t list_i[kWaves][kSliceListMax];
  __shared__ float group_max[32];
  __shared__ uint32_t wave_cnt[kWaves];
  __shared__ double wave_sum[kWaves];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t id = first_slice + blockIdx.x;
  // sequence of this slice: the last b whose first slice is not past it
  int b = 0;
  for (int step = 32; step > 0; step >>= 1)
    if (b + step < gt.batch && gt.scan_off[b + step] <= id) b += step;
  const int ns = gt.slices[b], n = gt.n[b], words = gt.words[b], vps = gt.slice_vecs[b];
  const int local = (int)(id - gt.scan_off[b]);  // 2^31 slices of a sequence would be 70 TB of logits
  const int row = local / ns, sl = local - row * ns;
  const int64_t first = gt.logit_off[b] + (int64_t)row * n;
  const auto [lead, v0, v1, have] = scan_slice(first, n, vps, sl);
  const float* p0 = a.logits + (first - lead) + 4 * (int64_t)v0;

  // float4 v holds entries 4 v - lead .. + 3 of the row; the last one of a row
  // may reach past its end and is read entry by entry.  The buffer ends with
  // the slice's whole float4s: loads past it return 0, which -inf replaces.
  // (The whole offset is the vector offset, which the range check is defined on.)
  f32x4 x[kScanVec];
  {
    constexpr int kNontemporal = 2;  // the nt bit of a buffer instruction's cache policy
    const __amdgpu_buffer_rsrc_t src =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p0), (short)0, have * 16, 0x00020000);
#pragma unroll
    for (int j = 0; j < kScanVec; ++j) {
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 y = __builtin_amdgcn_raw_buffer_load_b128(src, scan_offset(tid, j), 0, kNontemporal);
      x[j] = __builtin_bit_cast(f32x4, y);
    }
  }
  if (have < kGoldenSliceVecs) {  // uniform
    const int left = n + lead - 4 * (v0 + have);  // entries of the row past them, in this slice if have < v1 - v0
    const float* p = p0 + 4 * have;
    f32x4 last = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    if (have < v1 - v0) {
      last.x = p[0];
      if (left > 1) last.y = p[1];
      if (left > 2) last.z = p[2];
    }
#pragma unroll
    for (int j = 0; j < kScanVec; ++j) {
      const int v = tid + kThreads * j;
      if (v >= have) x[j] = v == have ? last : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
  }
  if (v0 == 0 && tid == 0) {  // entries before the row
    if (lead > 0) x[0].x = -INFINITY;
    if (lead > 1) x[0].y = -INFINITY;
    if (lead > 2) x[0].z = -INFINITY;
  }

  // maxima of 16-lane groups, 512 entries each
  float gm = -INFINITY;
#pragma unroll
  for (int j = 0; j < kScanVec; ++j) gm = max3(max3(x[j].x, x[j].y, gm), x[j].z, x[j].w);
  gm = fmax2(gm, dpp<kXor1>(gm));
  gm = fmax2(gm, dpp<kXor2>(gm));
  gm = fmax2(gm, dpp<kHalfMirror>(gm));
  gm = fmax2(gm, dpp<kMirror>(gm));
  if ((lane & 15) == 0) group_max[tid >> 4] = gm;
  lds_barrier();
  // lane i: the maximum over 1, 2, 4, 8, 16 groups around group i % 32, and the
  // smallest of those for the level; m, the slice's maximum
  const int cap = slice_cap(words, ns);
  const float y1 = group_max[lane & 31];
  const float y2 = fmax2(y1, dpp<kXor1>(y1));
  const float y4 = fmax2(y2, dpp<kXor2>(y2));
  const float y8 = fmax2(y4, dpp<kHalfMirror>(y4));
  const float y16 = fmax2(y8, dpp<kMirror>(y8));
  const float m = with16(y16, fmax2);
  // Entries at or above the threshold are listed, the others summed: exp(x - m)
  // as 2^(x c + off) with c = log2 e and off = -m c, each rounded to float32.
  const float off = slice_off(m);
  // the first level whose usual number of listed entries (130, 54, 22, 8, 3) fits
  int level = cap >= 200 ? 0 : cap >= 100 ? 1 : cap >= 44 ? 2 : cap >= 16 ? 3 : 4;
  float th;
  uint32_t before, count, mine;
  for (;; ++level) {
    th = level == 0 ? y1 : level == 1 ? y2 : level == 2 ? y4 : level == 3 ? y8 : y16;
    th = fmin2(th, dpp<kXor1>(th));
    th = fmin2(th, dpp<kXor2>(th));
    th = fmin2(th, dpp<kHalfMirror>(th));
    th = fmin2(th, dpp<kMirror>(th));
    th = level > 4 ? INFINITY : with16(th, fmin2);
    // (opaque copies, so that nothing is held in registers across the loop)
    float th2 = th;
    uint32_t e0 = 4u * (uint32_t)tid;
    asm volatile("" : "+v"(th2), "+v"(e0));
    mine = 0u;
#pragma unroll
    for (int j = 0; j < kScanVec; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t bal = __ballot(x[j][i] >= th2);
        if (bal != 0ull) {  // wave-uniform
          const uint32_t at = mine + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
          if (x[j][i] >= th2 && at < (uint32_t)kSliceListMax) {
            list_x[wave][at] = x[j][i];
            list_i[wave][at] = (uint16_t)(e0 + (uint32_t)(4 * kThreads * j + i));
          }
          mine += (uint32_t)__popcll(bal);
        }
      }
    }
    if (lane == 0) wave_cnt[wave] = mine;
    lds_barrier();
    before = count = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_cnt[w]);
      before += w < wave ? c : 0u;
      count += c;
    }
    if (count <= (uint32_t)cap) break;  // uniform; always at level 5, which lists nothing
    if (th == m) level = 4;  // every further threshold is m too (a slice of equal entries, masked ones for example)
    lds_barrier();
  }
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < kScanVec; ++j) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float w = __builtin_amdgcn_exp2f(__builtin_fmaf(x[j][i], kSliceLog2e, off));
      acc[i] += x[j][i] >= th ? 0.f : w;
    }
  }
  double sum = ((double)acc[0] + (double)acc[1]) + ((double)acc[2] + (double)acc[3]);
  sum = wave_reduce(sum, [](double p, double q) { return p + q; });
  if (lane == 0) wave_sum[wave] = sum;
  uint32_t* dst = a.bits + gt.bit_off[b] + (int64_t)row * words + (int64_t)sl * slice_words(words, ns);
  uint16_t* ids = reinterpret_cast<uint16_t*>(dst + kSliceHead + cap);
  for (uint32_t i = lane; i < mine; i += 64) {
    dst[kSliceHead + before + i] = __float_as_uint(list_x[wave][i]);
    ids[before + i] = list_i[wave][i];
  }
  lds_barrier();
  if (tid == 0) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += wave_sum[w];
    dst[0] = __float_as_uint(m);
    dst[1] = level > 4 ? key_of(m) + 1u : key_of(th);
    dst[2] = __float_as_uint((float)s);
    dst[3] = count;
  }
}

// The label bitmap and golden-set sizes start at zero (the vote kernel runs
// later): by the first launch of one workgroup per row.
__device__ __forceinline__ void zero_labels(const GoldenTable& gt, const GoldenArgs& a, int threads) {
  const int64_t i0 = (int64_t)blockIdx.x * threads + threadIdx.x, stride = (int64_t)gridDim.x * threads;
  for (int64_t i = i0; i < a.label_words; i += stride) a.label_bits[i] = 0u;
  if (a.golden_count != nullptr)
    for (int64_t i = i0; i < (int64_t)gt.batch * a.tau; i += stride) a.golden_count[i] = 0;
}

// Mark of a scanned row that the row kernel leaves open, in word kOpenWord of
// its bitmap.
constexpr uint32_t kOpenRow = 0x9E3779B9u;

constexpr int kRowThreads = 256;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kRowBins = 1024;  // bins of the one histogram over the listed keys
constexpr int kRowBinsPerThread = kRowBins / kRowThreads;
constexpr int kFew = 64;        // entries of the threshold bin resolved by rank in one wavefront
constexpr int kLdsWords = 2048; // bitmap words assembled at a time

// Bound: latency (1,344 rows of about 1,000 listed entries take 27 us).  Six
// 256-thread workgroups per CU (80 registers, 25 KiB of LDS), so that all of
// those rows are in flight at once; with 33 KiB and four per CU it took 35 us.
__global__ void __launch_bounds__(kRowThreads, 6)
golden_row_kernel(GoldenTable gt, GoldenArgs a) {
  __shared__ uint32_t lkey[kGoldenListMax], lidx[kGoldenListMax];
  __shared__ __align__(16) uint32_t lbm[kLdsWords];  // the histogram first, then the bitmap
  __shared__ uint32_t few_key[kFew];
  __shared__ uint64_t few_q[kFew];
  __shared__ uint64_t red[4][kRowWaves];
  __shared__ uint32_t sh_list, sh_few, sh_digit, sh_flag;
  __shared__ uint64_t sh_above;
  unsigned long long* hist = reinterpret_cast<unsigned long long*>(lbm);
  static_assert(kRowBins * 8 <= kLdsWords * 4 && kGoldenListMax <= kLdsWords, "shared areas");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  zero_labels(gt, a, kRowThreads);
  const int rows_per_seq = a.tau * a.layers;
  const int b = blockIdx.x / rows_per_seq, row = blockIdx.x % rows_per_seq;
  const int n = gt.n[b], words = gt.words[b], ns = gt.slices[b];
  if (ns == 0) return;  // a row that the exact kernel decides (the whole workgroup)
  uint32_t* bm = a.bits + gt.bit_off[b] + (int64_t)row * words;
  const uint64_t num = (uint64_t)a.p_num, den = (uint64_t)a.p_den;

  // ---- the listed entries of the row's slices (key 0: none; no finite logit
  // maps to it)
  constexpr int kPer = kGoldenSlots / kRowThreads;
  static_assert(kGoldenListMax <= kGoldenSlots, "slots");
  uint32_t key[kPer], ids[kPer / 2];  // ids: entry numbers within the slice, two to a word
  uint32_t mk = 0u, kth = 0u;  // largest key; entries with keys at or above kth are all listed
  float hm = 0.f, hsum = 0.f;  // header of slice tid
  const int sw = slice_words(words, ns), vps = gt.slice_vecs[b];
  const int cap = slice_cap(words, ns);
  const uint32_t inv = slot_inverse((uint32_t)cap);
  const int lead = (int)((gt.logit_off[b] + (int64_t)row * n) & 3);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t f = (uint32_t)(tid + j * kRowThreads), s = slot_slice(f, inv), i = f - s * (uint32_t)cap;
    uint32_t v = 0u, id = 0u, c = 0u;
    if ((int)s < ns) {
      const uint32_t* src = bm + (int64_t)s * sw;
      c = src[3];
      v = src[kSliceHead + i];
      id = reinterpret_cast<const uint16_t*>(src + kSliceHead + cap)[i];
    }
    key[j] = i < c ? key_of(__uint_as_float(v)) : 0u;
    ids[j / 2] = j % 2 ? ids[j / 2] | (id << 16) : id;
  }
  if (tid < ns) {
    const uint32_t* src = bm + (int64_t)tid * sw;
    hm = __uint_as_float(src[0]);
    mk = key_of(hm);
    kth = src[1];
    hsum = __uint_as_float(src[2]);
  }
  for (int s = tid + kRowThreads; s < ns; s += kRowThreads) {  // rows of over 2^20 entries
    mk = max(mk, key_of(__uint_as_float(bm[(int64_t)s * sw])));
    kth = max(kth, bm[(int64_t)s * sw + 1]);
  }
#pragma unroll
  for (int i = 0; i < kRowBins / kRowThreads; ++i) hist[tid + i * kRowThreads] = 0ull;
  if (tid == 0) sh_list = sh_few = sh_flag = 0u;
  mk = wave_reduce(mk, [](uint32_t p, uint32_t q) { return max(p, q); });
  kth = wave_reduce(kth, [](uint32_t p, uint32_t q) { return max(p, q); });
  if (lane == 0) red[0][wave] = ((uint64_t)mk << 32) | kth;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kRowWaves; ++w) {
    mk = max(mk, (uint32_t)(red[0][w] >> 32));
    kth = max(kth, (uint32_t)red[0][w]);
  }
  const float m = logit_of(mk);

  // ---- exact masses of the listed entries; the others' mass lies in an
  // interval.  Entries at or above kth go to the candidate list; those below
  // count in the total, but not every entry of their rank is listed.
  uint64_t all = 0ull, sel = 0ull;
  uint32_t low = 0xFFFFFFFFu;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (__ballot(key[j] != 0u) == 0ull) continue;  // wave-uniform
    const uint64_t q = key[j] ? mass_of(logit_of(key[j]), m) : 0ull;
    const bool in = key[j] >= kth && key[j] != 0u;
    all += q;
    sel += in ? q : 0ull;
    const uint64_t bal = __ballot(in);
    if (bal) {
      uint32_t at = 0u;
      if (lane == 0) at = atomicAdd(&sh_list, (uint32_t)__popcll(bal));
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
           __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
      if (in && at < (uint32_t)kGoldenListMax) {
        lkey[at] = key[j];
        const uint32_t id = j % 2 ? ids[j / 2] >> 16 : ids[j / 2] & 0xFFFFu;
        lidx[at] = slice_entry(slot_slice((uint32_t)(tid + j * kRowThreads), inv), vps, id, lead);
        low = min(low, key[j]);
      }
    }
  }
  double rest = 0.0, err = 0.0;
  auto add_slice = [&](float hm_, float hsum_) {
    if (slice_weightless((double)hm_, (double)m)) return;
    // no sum where no entry is left (not so for NaN, nor where the scale's own
    // rounding may have made every weight underflow: that leaves the row open)
    if (hsum_ <= 0.f && slice_error((double)hm_, (double)m, 0.0) < 1.0) return;
    // the weights' scale is 2^off, not the maximum
    const double R = (double)hsum_ * exp(-(double)slice_off(hm_) * 0.69314718055994530942 - (double)m);
    rest += R;
    err += R * slice_error((double)hm_, (double)m, fmax(log((double)(4 * vps) / (double)hsum_), 0.0));
  };
  if (tid < ns) add_slice(hm, hsum);
  for (int s = tid + kRowThreads; s < ns; s += kRowThreads)
    add_slice(__uint_as_float(bm[(int64_t)s * sw]), __uint_as_float(bm[(int64_t)s * sw + 2]));
  all = wave_reduce(all, [](uint64_t p, uint64_t r) { return p + r; });
  sel = wave_reduce(sel, [](uint64_t p, uint64_t r) { return p + r; });
  low = wave_reduce(low, [](uint32_t p, uint32_t r) { return min(p, r); });
  // (the slices' headers sit in the first ns threads)
  if (64 * wave < ns) {
    rest = wave_reduce(rest, [](double p, double r) { return p + r; });
    err = wave_reduce(err, [](double p, double r) { return p + r; });
  }
  __syncthreads();  // red[0]
  if (lane == 0) {
    red[0][wave] = all;
    red[1][wave] = sel;
    red[2][wave] = (uint64_t)__double_as_longlong(rest);
    red[3][wave] = (uint64_t)__double_as_longlong(err);
    atomicMax(&sh_flag, ~low);
  }
  __syncthreads();
  all = sel = 0ull;
  rest = err = 0.0;
#pragma unroll
  for (int w = 0; w < kRowWaves; ++w) {
    all += red[0][w];
    sel += red[1][w];
    rest += __longlong_as_double((long long)red[2][w]);
    err += __longlong_as_double((long long)red[3][w]);
  }
  low = ~sh_flag;  // the smallest candidate key
  const int nl = (int)sh_list;
  u128 need_lo, need_hi;
  bool fast = nl > 0 && nl <= kGoldenListMax;
  {
    // (and one unit per entry for the floor of the masses)
    constexpr double kUnit = 1099511627776.0;  // 2^40
    const double slack = err * kUnit + 8.0;
    const double r = rest * kUnit;
    fast = fast && r + slack < 4.0e18;  // not so for a sum past the range (NaN included)
    const uint64_t rhi = fast ? (uint64_t)(r + slack) + 1ull : 0ull;
    const double least = r - slack - (double)n;
    const uint64_t rlo = fast && least > 0.0 ? (uint64_t)least : 0ull;
    need_lo = mul64(all + rlo, num);
    need_hi = mul64(all + rhi, num);
    fast = fast && ge128(mul64(sel, den), need_hi);
  }

  // ---- the bin of the candidates' keys where the mass reaches p, then the
  // entries in it by rank (or its 1,024 sub-bins, when it holds more than
  // kFew).  Every decision below is uniform.
  uint32_t T = 0u, ties = 0u, r = 0u;
  uint32_t base = low, top = mk;  // the range of keys the threshold lies in
  uint64_t over = 0ull;           // mass of the candidates above it
  while (fast) {
    const uint32_t span = top - base;
    const int shift = span >> 10 ? 32 - __builtin_clz(span) - 10 : 0;
    for (int i = tid; i < nl; i += kRowThreads)
      if (lkey[i] >= base && lkey[i] <= top)
        atomicAdd(&hist[(lkey[i] - base) >> shift], (unsigned long long)mass_of(logit_of(lkey[i]), m));
    __syncthreads();
    // descending: thread t owns the bins below 1023 - kRowBinsPerThread t
    uint64_t mine[kRowBinsPerThread], mine_sum = 0ull;
#pragma unroll
    for (int j = 0; j < kRowBinsPerThread; ++j) {
      mine[j] = hist[kRowBins - 1 - kRowBinsPerThread * tid - j];
      mine_sum += mine[j];
    }
    uint64_t incl = mine_sum;
    int from = lane;  // (opaque, as in wave_reduce)
    asm volatile("" : "+v"(from));
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t y = __shfl(incl, from - off);
      if (lane >= off) incl += y;
    }
    if (lane == 63) red[0][wave] = incl;
    if (tid == 0) sh_flag = 0u;
    __syncthreads();
    uint64_t ex = over + incl - mine_sum;
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) ex += w < wave ? red[0][w] : 0ull;
#pragma unroll
    for (int j = 0; j < kRowBinsPerThread; ++j) {
      if (!ge128(mul64(ex, den), need_hi) && ge128(mul64(ex + mine[j], den), need_hi)) {
        sh_digit = (uint32_t)(kRowBins - 1 - kRowBinsPerThread * tid - j);
        sh_above = ex;
        sh_flag = 1u;
      }
      ex += mine[j];
    }
    __syncthreads();
    if (sh_flag == 0u) {  // no crossing (a logit that is not finite)
      fast = false;
      break;
    }
    base += sh_digit << shift;
    top = base + ((1u << shift) - 1u);
    over = sh_above;
    for (int i = tid; i < nl; i += kRowThreads) {
      if (lkey[i] >= base && lkey[i] <= top) {
        const uint32_t at = atomicAdd(&sh_few, 1u);
        if (at < (uint32_t)kFew) {
          few_key[at] = lkey[i];
          few_q[at] = mass_of(logit_of(lkey[i]), m);
        }
      }
    }
    __syncthreads();
    const int nf = (int)sh_few;
    if (nf > kFew && shift > 0) {
      __syncthreads();  // sh_few and the histogram start again
      if (tid == 0) sh_few = 0u;
#pragma unroll
      for (int i = 0; i < kRowBins / kRowThreads; ++i) hist[tid + i * kRowThreads] = 0ull;
      __syncthreads();
      continue;
    }
    // lane i: entry i of the bin, the mass above it, and how many equal it (a
    // bin of one key: every lane stands for that key)
    const bool one = nf > kFew;
    const uint32_t fk = one ? base : lane < nf ? few_key[lane] : 0u;
    const uint64_t qT = one ? few_q[0] : lane < nf ? few_q[lane] : 0ull;
    uint64_t above = over;
    ties = one ? (uint32_t)nf : 0u;
    for (int i = 0; i < nf && !one; ++i) {
      above += few_key[i] > fk ? few_q[i] : 0ull;
      ties += few_key[i] == fk ? 1u : 0u;
    }
    const uint64_t hit = __ballot((one || lane < nf) && !ge128(mul64(above, den), need_hi) &&
                                  ge128(mul64(above + (uint64_t)ties * qT, den), need_hi));
    if (hit == 0ull) {
      fast = false;
      break;
    }
    // the fewest entries equal to T that reach the mass (1 .. ties)
    uint32_t lo = 1, hi = ties;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) / 2;
      if (ge128(mul64(above + (uint64_t)mid * qT, den), need_hi)) hi = mid;
      else lo = mid + 1;
    }
    // settled when one entry less stays short of p at the other end too
    const bool sure = !ge128(mul64(above + (uint64_t)(lo - 1u) * qT, den), need_lo);
    const int first = __builtin_ctzll(hit);
    T = (uint32_t)__builtin_amdgcn_readlane((int)fk, first);
    r = (uint32_t)__builtin_amdgcn_readlane((int)lo, first);
    ties = (uint32_t)__builtin_amdgcn_readlane((int)ties, first);
    // (otherwise the boundary falls inside the interval: about one row in 10,000)
    fast = __builtin_amdgcn_readlane((int)sure, first) != 0;
    break;
  }
  if (!fast) {  // golden_exact_kernel decides this row
    if (tid == 0) bm[kOpenWord] = kOpenRow;
    return;
  }

  // ---- members: candidates above T, and the r entries equal to T with the lowest ids
  const bool some = r != ties;
  int t0 = tid;  // (opaque, as in wave_reduce)
  asm volatile("" : "+v"(t0));
  for (int w0 = 0; w0 < words; w0 += kLdsWords) {
    const int nw = min(words - w0, kLdsWords);
    __syncthreads();
    for (int w = t0; w < nw; w += kRowThreads) lbm[w] = 0u;
    __syncthreads();
    for (int i = t0; i < nl; i += kRowThreads) {
      const uint32_t k = lkey[i], e = lidx[i];
      bool in = k >= T;
      if (some && k == T) {
        uint32_t rank = 0u;
        for (int j = 0; j < nl; ++j) rank += lkey[j] == T && lidx[j] < e ? 1u : 0u;
        in = rank < r;
      }
      const int w = (int)(e >> 5) - w0;
      if (in && w >= 0 && w < nw) atomicOr(&lbm[w], 1u << (e & 31u));
    }
    __syncthreads();
    // (a bitmap that happens to hold the mark of an open row there is left to
    // the exact kernel, whose result is the same)
    if (w0 == 0 && lbm[kOpenWord] == kOpenRow) {
      if (tid == 0) bm[kOpenWord] = kOpenRow;
      return;
    }
    for (int w = t0; w < nw; w += kRowThreads) bm[w0 + w] = lbm[w];
  }
  if (a.nucleus_size != nullptr) {
    uint32_t n_in = 0u;
    for (int i = t0; i < nl; i += kRowThreads) n_in += lkey[i] > T ? 1u : 0u;
    n_in = wave_reduce(n_in, [](uint32_t p, uint32_t s) { return p + s; });
    if (lane == 0) red[1][wave] = n_in;
    __syncthreads();
    if (tid == 0) {
      uint32_t total = r;
#pragma unroll
      for (int w = 0; w < kRowWaves; ++w) total += (uint32_t)red[1][w];
      a.nucleus_size[(int64_t)b * rows_per_seq + row] = (int32_t)total;
    }
  }
}

// Shared arrays of the exact decision.  The histogram is done with before the
// first candidate is staged, and the digit rounds use its first kSubBins bins:
// the candidates take the space of the others.
struct ExactLds {
  unsigned long long hist[kBins];
  uint32_t sub_cnt[kSubBins];
  uint64_t wave_tot[kWaves];
  uint32_t wave_mk[kWaves];
  uint32_t sh_cnt, sh_digit;
  uint64_t sh_above;
};

// The exact decision of one row by a workgroup.  HOLD > 0: the row (at most
// HOLD * kThreads entries) is read once and held in registers, HOLD entries per
// thread; HOLD = 0: it is read in every pass.  mk: the key of the row's maximum,
// or of this thread's share of it; 0 (HOLD > 0) where the held entries tell.
template <int HOLD>
__device__ __forceinline__ void exact_row(const GoldenArgs& a, ExactLds& L, const float* S, uint32_t* bm, int n, int words,
                                          int32_t* size_out, uint32_t mk) {
  unsigned long long* hist = L.hist;
  uint32_t* sub_cnt = L.sub_cnt;
  uint32_t* cand_key = reinterpret_cast<uint32_t*>(hist + kSubBins);
  uint32_t* cand_idx = cand_key + kCand;
  static_assert(kSubBins + kCand <= kBins, "shared areas");
  uint64_t* wave_tot = L.wave_tot;
  uint32_t &sh_cnt = L.sh_cnt, &sh_digit = L.sh_digit;
  uint64_t& sh_above = L.sh_above;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // The round at `base` gives this lane the entries base + e0 + 64 u: 64
  // consecutive entries per wavefront load, kUnroll consecutive groups per
  // wavefront.  Buffer loads past the row's end return 0, which -inf replaces.
  constexpr int kUnroll = HOLD > 0 && HOLD < 16 ? HOLD : 16;
  constexpr int kRound = kThreads * kUnroll;
  int e0 = wave * kUnroll * 64 + lane;
  float held[HOLD > 0 ? HOLD : 1];
  const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(S), (short)0, n * 4, 0x00020000);
  auto load = [&](int base, float* v, bool last) {
    constexpr int kNontemporal = 2;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int at = 4 * (base + e0) + 256 * u;
      v[u] = __uint_as_float(last ? __builtin_amdgcn_raw_buffer_load_b32(src, at, 0, kNontemporal)
                                  : __builtin_amdgcn_raw_buffer_load_b32(src, at, 0, 0));
    }
    if (base + kRound > n) {  // uniform
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) v[u] = e0 < n - base - 64 * u ? v[u] : -INFINITY;
    }
  };
  auto rounds = [&](bool last, auto&& f) {
    if constexpr (HOLD > 0) {
      // (opaque, so that no pass keeps what it derives from them for the next)
      asm volatile("" : "+v"(e0));
#pragma unroll
      for (int i = 0; i < HOLD; ++i) asm volatile("" : "+v"(held[i]));
#pragma unroll
      for (int r = 0; r < HOLD / kUnroll; ++r)
        if (r * kRound < n) f(r * kRound, held + r * kUnroll);  // uniform
    } else {
      for (int base = 0; base < n; base += kRound) {
        float v[kUnroll];
        load(base, v, last);
        f(base, v);
      }
    }
  };
  if constexpr (HOLD > 0) {
#pragma unroll
    for (int r = 0; r < HOLD / kUnroll; ++r)
      if (r * kRound < n) load(r * kRound, held + r * kUnroll, true);
    if (mk == 0u) {
      float mx = -INFINITY;
      rounds(false, [&](int, const float* v) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) mx = fmaxf(mx, v[u]);
      });
      mk = key_of(mx);
    }
  }
  mk = wave_reduce(mk, [](uint32_t p, uint32_t q) { return max(p, q); });
  if (lane == 0) L.wave_mk[wave] = mk;
  for (int i = tid; i < kBins; i += kThreads) hist[i] = 0ull;
  if (tid == 0) sh_cnt = 0u;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mk = max(mk, L.wave_mk[w]);
  const float m = logit_of(mk);

  // ---- first pass: mass histogram by the top 12 bits of the order key
  rounds(false, [&](int, const float* v) {
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint64_t q = mass_of(v[u], m);  // 0 past the end
      if (q) atomicAdd(&hist[key_of(v[u]) >> 20], (unsigned long long)q);
    }
  });
  __syncthreads();

  // descending scan of the bins: thread t owns the kBinsPerThread bins below
  // kBins - 1 - kBinsPerThread * t
  uint64_t own_sum = 0;
#pragma unroll
  for (int j = 0; j < kBinsPerThread; ++j) own_sum += hist[kBins - 1 - kBinsPerThread * tid - j];
  uint64_t Z;
  uint64_t before = block_scan_u64(own_sum, wave_tot, &Z);
  const u128 need = mul64(Z, (uint64_t)a.p_num);
  const uint64_t den = (uint64_t)a.p_den;
  if (!ge128(mul64(before, den), need) && ge128(mul64(before + own_sum, den), need)) {  // one thread
    for (int j = 0; j < kBinsPerThread; ++j) {
      const uint64_t own = hist[kBins - 1 - kBinsPerThread * tid - j];
      if (ge128(mul64(before + own, den), need)) {
        sh_digit = (uint32_t)(kBins - 1 - kBinsPerThread * tid - j);
        sh_above = before;
        break;
      }
      before += own;
    }
  }
  __syncthreads();
  const uint32_t bstar = sh_digit;
  uint64_t above = sh_above;  // mass of every key above the current prefix

  // ---- second pass: bitmap of the bins above bstar, entries of bstar to LDS
  const float bin_start = logit_of(bstar << 20), bin_end = logit_of((bstar + 1u) << 20);
  uint32_t n_in = 0;
  rounds(true, [&](int base, const float* v) {
    // the wavefront's kUnroll groups are 2 * kUnroll consecutive bitmap
    // words; lane u < kUnroll collects the two of group u and stores them.
    // (The bins' bounds as logits: a comparison is a ballot.  No finite logit's
    // bin is as low as that of -inf past the end.)
    uint64_t word = 0u;
    int l = lane;  // (opaque: the masks of its comparisons would not fit the scalar registers)
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint64_t in = __ballot(v[u] >= bin_end);
      const uint64_t cnd = __ballot(v[u] >= bin_start) & ~in;
      word = l == u ? in : word;
      n_in += (uint32_t)__popcll(in);
      if (cnd) {  // wave-uniform
        uint32_t first = 0;
        if (lane == 0) first = atomicAdd(&sh_cnt, (uint32_t)__popcll(cnd));
        first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
        if ((cnd >> lane) & 1ull) {
          const uint32_t pos = first + __builtin_amdgcn_mbcnt_hi((uint32_t)(cnd >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)cnd, 0u));
          if (pos < kCand) {
            cand_key[pos] = key_of(v[u]);
            cand_idx[pos] = (uint32_t)(base + e0 + 64 * u);
          }
        }
      }
    }
    const int w = (base >> 5) + wave * 2 * kUnroll + 2 * lane;
    if (lane < kUnroll && w < words) {
      bm[w] = (uint32_t)word;
      if (w + 1 < words) bm[w + 1] = (uint32_t)(word >> 32);
    }
  });
  if (lane == 0) wave_tot[wave] = n_in;
  __syncthreads();
  uint32_t count_in = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) count_in += (uint32_t)wave_tot[w];
  const uint32_t nc = sh_cnt;
  const bool staged = nc <= (uint32_t)kCand;
  __syncthreads();  // wave_tot and sh_cnt are reused below

  // ---- a bin of few entries: an entry is in the set when the mass before it
  // (of larger keys, and of equal keys with lower ids) falls short of p.  Every
  // entry is compared with every other, by 8 threads; with 150 entries that is
  // no faster than the digits below (8,192 flat entries 63 us against 61), with
  // a handful it takes half their time (8,192 peaked ones 43 -> 36).
  if (nc <= (uint32_t)kFewCand) {  // uniform
    if (tid < (int)nc) hist[tid] = mass_of(logit_of(cand_key[tid]), m);
    __syncthreads();
    constexpr int kShare = kThreads / kFewCand;
    const uint32_t i = (uint32_t)tid / kShare;
    auto order = [&](uint32_t j) { return ((uint64_t)cand_key[j] << 32) | (uint32_t)~cand_idx[j]; };
    const uint64_t mine = i < nc ? order(i) : ~0ull;
    uint64_t ahead = 0ull;
    for (uint32_t j = (uint32_t)tid % kShare; j < nc; j += kShare) ahead += order(j) > mine ? hist[j] : 0ull;
#pragma unroll
    for (int off = 1; off < kShare; off *= 2) ahead += __shfl_xor(ahead, off);
    const bool in = i < nc && tid % kShare == 0 && !ge128(mul64(above + ahead, den), need);
    if (in) {
      const uint32_t e = cand_idx[i];
      atomicOr(&bm[e >> 5], 1u << (e & 31));
    }
    if (size_out == nullptr) return;
    const uint64_t bal = __ballot(in);
    if (lane == 0) wave_tot[wave] = (uint64_t)__popcll(bal);
    __syncthreads();
    if (tid == 0) {
      uint32_t tot = count_in;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) tot += (uint32_t)wave_tot[w];
      *size_out = (int32_t)tot;
    }
    return;
  }

  // the entries whose key has the given prefix: staged ones, or the row
  auto each = [&](uint32_t prefix, int shift, auto&& f) {
    if (staged) {
      for (uint32_t i = tid; i < nc; i += kThreads) {
        const uint32_t key = cand_key[i];
        if ((key >> shift) == prefix) f(key, cand_idx[i]);
      }
    } else {
      for (int e = tid; e < n; e += kThreads) {
        const uint32_t key = key_of(S[e]);
        if ((key >> shift) == prefix) f(key, (uint32_t)e);
      }
    }
  };

  // ---- two 10-bit digits inside the threshold bin
  uint32_t prefix = bstar;
  for (int round = 0; round < 2; ++round) {
    const int shift = 10 - 10 * round;  // digit bits [shift, shift + 10)
    for (int i = tid; i < kSubBins; i += kThreads) {
      hist[i] = 0ull;
      sub_cnt[i] = 0u;
    }
    __syncthreads();
    each(prefix, shift + 10, [&](uint32_t key, uint32_t) {
      const uint32_t d = (key >> shift) & (kSubBins - 1);
      atomicAdd(&hist[d], (unsigned long long)mass_of(logit_of(key), m));
      atomicAdd(&sub_cnt[d], 1u);
    });
    __syncthreads();
    // descending: thread t owns the kSubPerThread digits below 1023 - kSubPerThread * t
    uint64_t mine[kSubPerThread], mine_sum = 0;
#pragma unroll
    for (int j = 0; j < kSubPerThread; ++j) {
      mine[j] = hist[kSubBins - 1 - kSubPerThread * tid - j];
      mine_sum += mine[j];
    }
    uint64_t tot;
    uint64_t ex = above + block_scan_u64(mine_sum, wave_tot, &tot);
#pragma unroll
    for (int j = 0; j < kSubPerThread; ++j) {
      const int d = kSubBins - 1 - kSubPerThread * tid - j;
      if (sub_cnt[d] != 0u && !ge128(mul64(ex, den), need) && ge128(mul64(ex + mine[j], den), need)) {
        sh_digit = (uint32_t)d;
        sh_above = ex;
      }
      ex += mine[j];
    }
    __syncthreads();
    prefix = (prefix << 10) | sh_digit;
    above = sh_above;
  }
  const uint32_t T = prefix;
  const uint32_t ties = sub_cnt[T & (kSubBins - 1)];
  const uint64_t qT = mass_of(logit_of(T), m);
  // the fewest entries equal to T that reach the mass (1 .. ties)
  uint32_t lo = 1, hi = ties;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) / 2;
    if (ge128(mul64(above + (uint64_t)mid * qT, den), need)) hi = mid;
    else lo = mid + 1;
  }
  const uint32_t r = lo;

  // ---- the threshold bin's members: keys above T, and T itself when all of
  // its entries are needed
  uint32_t n_mid = 0;
  each(bstar, 20, [&](uint32_t key, uint32_t idx) {
    if (key > T || (key == T && r == ties)) {
      atomicOr(&bm[idx >> 5], 1u << (idx & 31));
      ++n_mid;
    }
  });
  if (r != ties && wave == 0) {
    // only r of the entries equal to T, the lowest indices first
    uint32_t run = 0;
    for (int g0 = 0; g0 < n && run < r; g0 += 64) {
      const int e = g0 + lane;
      const bool tie = e < n && key_of(S[e]) == T;
      const uint64_t bal = __ballot(tie);
      const uint32_t rank = run + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      if (tie && rank < r) atomicOr(&bm[e >> 5], 1u << (e & 31));
      run += (uint32_t)__popcll(bal);
    }
  }
  n_mid = wave_reduce(n_mid, [](uint32_t x, uint32_t y) { return x + y; });
  __syncthreads();
  if (lane == 0) wave_tot[wave] = n_mid;
  __syncthreads();
  if (tid == 0 && size_out != nullptr) {
    uint32_t tot = count_in + (r == ties ? 0u : r);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) tot += (uint32_t)wave_tot[w];
    *size_out = (int32_t)tot;
  }
}

// Rows that are not scanned, and the scanned rows that the row kernel left open.
__global__ void __launch_bounds__(kThreads, 6)
golden_exact_kernel(GoldenTable gt, GoldenArgs a) {
  __shared__ ExactLds L;
  const int tid = threadIdx.x;
  const int rows_per_seq = a.tau * a.layers;
  const int b = blockIdx.x / rows_per_seq, row = blockIdx.x % rows_per_seq;
  const int n = gt.n[b], words = gt.words[b], ns = gt.slices[b];
  if (gt.scan_off[gt.batch] == 0) zero_labels(gt, a, kThreads);
  const float* S = a.logits + gt.logit_off[b] + (int64_t)row * n;
  uint32_t* bm = a.bits + gt.bit_off[b] + (int64_t)row * words;
  int32_t* size = a.nucleus_size == nullptr ? nullptr : a.nucleus_size + (int64_t)b * rows_per_seq + row;
  if (ns == 0) {
    if (n <= 8 * kThreads) exact_row<8>(a, L, S, bm, n, words, size, 0u);
    else exact_row<kGoldenHeld>(a, L, S, bm, n, words, size, 0u);
    return;
  }
  if (bm[kOpenWord] != kOpenRow) return;  // the whole workgroup
  // the row's maximum is the largest of its slices'
  uint32_t mk = 0u;
  for (int sl = tid; sl < ns; sl += kThreads)
    mk = max(mk, key_of(__uint_as_float(bm[(int64_t)sl * slice_words(words, ns)])));
  exact_row<0>(a, L, S, bm, n, words, size, mk);
}

// Bit-sliced vote counters: c[k] holds bit k of the count of each of 32 entries.
constexpr int kCountBits = 7;  // counts up to 127 >= LSA_MAX_GOLDEN_LAYERS
// Steps per thread: with two, one OR into the label bitmap serves both, which pays
// once the bitmaps are long (4,096 words: 11.9 us with one step, 9.2 with two, 11.0
// with four; 1,024: 8.7, 6.0; 512: 6.3, 6.6; 32: 4.6, 6.7, as half the wavefronts
// take twice as long).
constexpr int kVoteTwoSteps = 768;  // words of the longest row from which a thread takes two steps
// Layers' words in flight at once; the last batch is padded.  4,096 words, 8, 21, 30,
// 48 and 61 layers, us: 8 in flight 6.3, 9.0, 10.5, 12.9, 15.7; 16 7.0, 9.3, 9.9,
// 12.8, 15.0; 24 8.2, 9.0, 12.0, 13.1, 16.0; 32 9.5, 9.5, 10.0, 14.7, 15.6.
constexpr int kVoteBatch = 16;

template <int kVoteSteps>
__global__ void __launch_bounds__(256)
golden_vote_kernel(GoldenTable gt, GoldenArgs a, uint32_t* __restrict__ label_bits, int32_t* golden_count) {
  __shared__ uint32_t cnt_sh[kVoteSteps];
  const int b = blockIdx.z, i0 = blockIdx.y * kVoteSteps;
  const int w = blockIdx.x * 256 + threadIdx.x;
  const int words = gt.words[b];
  if (blockIdx.x * 256 >= words) return;  // the whole workgroup
  if (threadIdx.x < kVoteSteps) cnt_sh[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t label = 0u;
  for (int i = i0; i < min(i0 + kVoteSteps, a.tau); ++i) {
    uint32_t A = 0u;
    if (w < words) {
      uint32_t c[kCountBits] = {};
      const uint32_t* src = a.bits + gt.bit_off[b] + (int64_t)i * a.layers * words + w;
      for (int l0 = 0; l0 < a.layers; l0 += kVoteBatch) {
        uint32_t x[kVoteBatch];
#pragma unroll
        for (int j = 0; j < kVoteBatch; ++j) x[j] = l0 + j < a.layers ? src[(int64_t)(l0 + j) * words] : 0u;
#pragma unroll
        for (int j = 0; j < kVoteBatch; ++j) {
          uint32_t carry = x[j];
#pragma unroll
          for (int k = 0; k < kCountBits; ++k) {
            const uint32_t t = c[k] & carry;
            c[k] ^= carry;
            carry = t;
          }
        }
      }
      // count >= theta, bit-sliced, from the most significant bit down
      uint32_t gt_ = 0u, eq = 0xFFFFFFFFu;
#pragma unroll
      for (int k = kCountBits - 1; k >= 0; --k) {
        if ((a.theta >> k) & 1) {
          eq &= c[k];
        } else {
          gt_ |= eq & c[k];
          eq &= ~c[k];
        }
      }
      A = gt_ | eq;
    }
    label |= A;
    if (golden_count != nullptr && __ballot(A != 0u) != 0ull) {
      uint32_t cnt = (uint32_t)__popc(A);
      cnt = wave_reduce(cnt, [](uint32_t x, uint32_t y) { return x + y; });
      if ((threadIdx.x & 63) == 0) atomicAdd(&cnt_sh[i - i0], cnt);
    }
  }
  if (label) atomicOr(&label_bits[gt.label_word_off[b] + w], label);
  if (golden_count != nullptr) {
    __syncthreads();
    if (threadIdx.x < kVoteSteps && cnt_sh[threadIdx.x] != 0u)
      atomicAdd(&golden_count[b * a.tau + i0 + threadIdx.x], (int32_t)cnt_sh[threadIdx.x]);
  }
}

// Rounds of up to 8 consecutive words per thread, held in registers between the
// count and the emission.  Short bitmaps are spread over all threads: a thread
// emits its entries one by one, and 32 words of dense labels took 11.8 us on
// four threads, 4.0 on 32.
__global__ void __launch_bounds__(kThreads)
golden_compact_kernel(GoldenTable gt, const uint32_t* __restrict__ label_bits, int32_t* labels,
                      int32_t* label_count) {
  constexpr int kPerMax = 8;
  __shared__ uint64_t wave_tot[kWaves];
  const int b = blockIdx.x, tid = threadIdx.x;
  const int words = gt.words[b];
  const uint32_t* src = label_bits + gt.label_word_off[b];
  const int per = min(kPerMax, (words + kThreads - 1) / kThreads);
  int32_t* out = labels + gt.entry_off[b];
  uint64_t base = 0;
  for (int r0 = 0; r0 < words; r0 += kThreads * per) {
    const int w0 = r0 + tid * per;
    uint32_t x[kPerMax];
    uint64_t cnt = 0;
#pragma unroll
    for (int j = 0; j < kPerMax; ++j) {
      x[j] = j < per && w0 + j < words ? src[w0 + j] : 0u;
      cnt += (uint64_t)__popc(x[j]);
    }
    uint64_t total;
    uint64_t pos = base + block_scan_u64(cnt, wave_tot, &total);
#pragma unroll
    for (int j = 0; j < kPerMax; ++j) {
      while (x[j]) {
        out[pos++] = 32 * (w0 + j) + __builtin_ctz(x[j]);
        x[j] &= x[j] - 1u;
      }
    }
    base += total;
  }
  if (tid == 0) label_count[b] = (int32_t)base;
}

}  // namespace

hipError_t launch_golden(const GoldenTable& gt, const GoldenArgs& a, uint32_t* label_bits, int64_t label_words,
                         int32_t* labels, int32_t* label_count, int32_t* golden_count, hipStream_t s) {
  GoldenArgs ra = a;
  ra.label_bits = label_bits;
  ra.label_words = label_words;
  ra.golden_count = golden_count;
  // a grid holds fewer than 2^32 threads
  for (int64_t first = 0; first < gt.scan_off[gt.batch]; first += kGoldenScanGrid)
    hipLaunchKernelGGL(golden_scan_kernel, dim3((unsigned)std::min<int64_t>(kGoldenScanGrid, gt.scan_off[gt.batch] - first)),
                       dim3(kThreads), 0, s, gt, ra, first);
  const dim3 rows((unsigned)(gt.batch * a.tau * a.layers));
  if (gt.scan_off[gt.batch] > 0) hipLaunchKernelGGL(golden_row_kernel, rows, dim3(kRowThreads), 0, s, gt, ra);
  hipLaunchKernelGGL(golden_exact_kernel, rows, dim3(kThreads), 0, s, gt, ra);
  int max_words = 0;
  for (int b = 0; b < gt.batch; ++b) max_words = std::max(max_words, gt.words[b]);
  const unsigned vote_x = (unsigned)((max_words + 255) / 256);
  if (max_words >= kVoteTwoSteps)
    hipLaunchKernelGGL(golden_vote_kernel<2>, dim3(vote_x, (unsigned)((a.tau + 1) / 2), (unsigned)gt.batch), dim3(256), 0,
                       s, gt, a, label_bits, golden_count);
  else
    hipLaunchKernelGGL(golden_vote_kernel<1>, dim3(vote_x, (unsigned)a.tau, (unsigned)gt.batch), dim3(256), 0, s, gt, a,
                       label_bits, golden_count);
  hipLaunchKernelGGL(golden_compact_kernel, dim3((unsigned)gt.batch), dim3(kThreads), 0, s, gt,
                     (const uint32_t*)label_bits, labels, label_count);
  return hipGetLastError();
}

}  // namespace lsa
