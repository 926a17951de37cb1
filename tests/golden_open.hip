// The golden-label scan and row kernels on their own, so that a test can see
// which rows they leave open: the library's next kernel overwrites the mark.
#include "../paper_2606_09079_amd/csrc/golden.hip"

// `rows` rows of n entries (one step), more than kGoldenDirectMax of them;
// `bits` holds rows * ceil(n / 32) words.
extern "C" int golden_scan_and_rows(const float* logits, int32_t n, int32_t rows, int32_t p_num, int32_t p_den,
                                    uint32_t* bits, void* stream) {
  using namespace lsa;
  if (n <= kGoldenDirectMax || n > LSA_MAX_GOLDEN_ENTRIES || rows < 1 || rows > LSA_MAX_GOLDEN_LAYERS) return -1;
  GoldenTable t = {};
  t.batch = 1;
  t.n[0] = n;
  t.words[0] = (n + 31) / 32;
  const GoldenSlices gs = golden_slices(n, 0);
  t.slices[0] = gs.slices;
  t.slice_vecs[0] = gs.slice_vecs;
  t.scan_off[1] = (int64_t)rows * gs.slices;
  GoldenArgs a = {};
  a.logits = logits;
  a.bits = bits;
  a.p_num = p_num;
  a.p_den = p_den;
  a.tau = 1;
  a.layers = rows;
  a.theta = 1;
  const auto s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(golden_scan_kernel, dim3((unsigned)t.scan_off[1]), dim3(kThreads), 0, s, t, a, (int64_t)0);
  hipLaunchKernelGGL(golden_row_kernel, dim3((unsigned)rows), dim3(kRowThreads), 0, s, t, a);
  return (int)hipGetLastError();
}
extern "C" int32_t golden_open_word() { return lsa::kOpenWord; }
extern "C" uint32_t golden_open_mark() { return lsa::kOpenRow; }
