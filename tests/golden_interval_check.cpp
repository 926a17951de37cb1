// The interval that stands for a slice's unlisted entries, against their exact
// integer masses: the scan's float32 sum is emulated with every approximation
// at its limit, over logits of both signs up to 1e9, spreads from one unit in
// the last place to 40, and row maxima up to 63 above the slice's.
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "golden_geometry.h"

using namespace lsa;

// exp(x), x <= 0, by the fixed float32 method that lsa.h documents
static float fixed_exp(float x) {
  if (x > 0.f) x = 0.f;
  if (x < -64.f) return 0.f;
  const float k = rintf(x * 1.44269502e+00f);
  float r = fmaf(-k, 6.9314575195e-01f, x);
  r = fmaf(-k, 1.4286067653e-06f, r);
  float p = 1.f / 5040.f;
  const float c[7] = {1.f / 720.f, 1.f / 120.f, 1.f / 24.f, 1.f / 6.f, 1.f / 2.f, 1.f, 1.f};
  for (float a : c) p = fmaf(p, r, a);
  return ldexpf(p, (int)k);
}

int main() {
  std::mt19937_64 rng(11);
  std::normal_distribution<double> gauss;
  double worst = 0.0;
  long tried = 0;
  const double mags[] = {0, 1, 30, 1e3, 1e5, 1e6, 3e6, 7e6, 1e7, 3e7, 1e8, 3e8, 1e9, 1e10, 1e15, 1e30, 3e38};
  const double spreads[] = {0, 1e-3, 0.1, 1, 4, 16, 40};
  const double aboves[] = {0, 0.5, 5, 30, 63};
  for (double mag : mags)
    for (int sign = -1; sign <= 1; sign += 2)
      for (double spread : spreads)
        for (double above : aboves)
          for (int n : {512, 2050, 16384}) {
            std::vector<float> x(n);
            for (auto& v : x) v = (float)(sign * mag + spread * gauss(rng));
            float m = x[0];
            for (float v : x) m = fmaxf(m, v);
            const float M = (float)((double)m + above);
            if (!((double)M - (double)m <= 64.0)) continue;  // (M rounded away)
            const float off = slice_off(m);
            // every entry unlisted: 32 partial sums a thread holds are added up in double
            for (double bias : {-2.4e-7, 2.4e-7}) {
              double sum = 0.0, exact = 0.0;
              for (int t = 0; t < n; t += 8) {
                float acc = 0.f;
                for (int i = t; i < t + 8 && i < n; ++i)
                  acc += (float)(exp2((double)fmaf(x[i], kSliceLog2e, off)) * (1.0 + bias));
                sum += (double)acc;
              }
              for (float v : x) exact += floor(ldexp((double)fixed_exp(v - M), 40));
              const float hsum = (float)sum;
              if (!(hsum > 0.f) || std::isinf(hsum)) {  // the sum says nothing, and the bound has to say so
                if (slice_error((double)m, (double)M, 0.0) < 1.0) {
                  printf("m=%g spread=%g: sum %g within a finite bound\n", (double)m, spread, (double)hsum);
                  return 1;
                }
                continue;
              }
              const double R = (double)hsum * exp(-(double)off * 0.69314718055994530942 - (double)M) * 0x1p40;
              const double d = fmax(log((double)n / (double)hsum), 0.0);
              const double err = slice_error((double)m, (double)M, d) * R + 8.0;
              ++tried;
              const double over = R - (double)n - err - exact, under = exact - (R + err);
              worst = fmax(worst, fabs(R - exact) / (err + (double)n));
              if (over > 0.0 || under > 0.0) {
                printf("m=%g spread=%g M-m=%g n=%d: sum %.17g exact %.17g bound %.3g\n", (double)m, spread, above, n, R,
                       exact, err);
                return 1;
              }
            }
          }
  // slices that lie so far below the row's maximum that they are left out have no mass
  const float lowest = -3.402823466e38f;
  for (float M : {-1e30f, -1e9f, -100.f, 0.f, 5.f, 1e9f, 3e38f})
    for (double below : {64.0 + 1e-5, 65.0, 1e4, 1e10, 1e30, 3.4e38}) {
      const double md = (double)M - below;
      const float m = md < (double)lowest ? lowest : (float)md;
      if (!slice_weightless((double)m, (double)M)) continue;
      ++tried;
      if (fixed_exp(m - M) * 0x1p40f >= 1.f) {
        printf("m=%g M=%g: an entry of a weightless slice has mass\n", (double)m, (double)M);
        return 1;
      }
    }
  if (!slice_weightless((double)lowest, -1e30) || slice_weightless(-64.0, 0.0)) return 1;
  printf("ok: %ld slices, largest error %.3f of its bound\n", tried, worst);
  return 0;
}
