// Host-only check of the margin that the refresh's check kernel deducts (csrc/fira_refresh.h, refresh_check_tolerance): columns
// whose bf16 remainders all have one sign or the largest size there is are taken through its arithmetic (planes h and m, products h m + m h, then h h, in
// sums of 32 rows) with fp32 additions that round to nearest and with ones that cut off, and must stay within the margin of their exact product.
// Built and run by tests/test_host_refresh_check.py.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "../paper_2410_01623_amd/csrc/fira_refresh.h"

namespace {

float bf16_nearest(float x) {          // (no NaN or infinity here)
  uint32_t u;
  std::memcpy(&u, &x, 4);
  u = (u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000u;
  std::memcpy(&x, &u, 4);
  return x;
}

// a + b in fp32: nearest, or cut off towards zero
float add(float a, double b, bool cut) {
  const double s = (double)a + b;
  float f = (float)s;
  if (cut && std::fabs((double)f) > std::fabs(s)) f = std::nextafterf(f, 0.0f);
  return f;
}

float as_the_kernel(const std::vector<float>& a, const std::vector<float>& b, bool cut) {
  float sum = 0.0f;
  for (size_t s0 = 0; s0 < a.size(); s0 += 32) {
    const size_t s1 = std::min(a.size(), s0 + 32);
    float part = 0.0f;
    for (int pass = 0; pass < 2; ++pass)
      for (size_t s = s0; s < s1; ++s) {
        const float ha = bf16_nearest(a[s]), hb = bf16_nearest(b[s]), ma = bf16_nearest(a[s] - ha), mb = bf16_nearest(b[s] - hb);
        if (pass) part = add(part, (double)ha * hb, cut);
        else part = add(add(part, (double)ha * mb, cut), (double)ma * hb, cut);
      }
    sum = add(sum, part, false);
  }
  return sum;
}

double exact(const std::vector<float>& a, const std::vector<float>& b) {
  long double d = 0.0L;
  for (size_t s = 0; s < a.size(); ++s) d += (long double)a[s] * b[s];
  return (double)d;
}

}  // namespace

int main() {
  const float done_tol = 1e-4f;
  std::mt19937_64 rng(7);
  std::uniform_real_distribution<double> uni(0.0, 1.0);
  int failures = 0;
  double used = 0.0;                   // largest share of the margin that a pair takes
  for (int S : {1, 31, 64, 232, 254, 970, 2048, 4096, 11008}) {
    const double margin = (double)done_tol - (double)refresh_check_tolerance(done_tol, S);
    for (int kind = 0; kind < 6; ++kind)
      for (int trial = 0; trial < 40; ++trial) {
        std::vector<float> a(S), b(S);
        // squared norm 1 + defect, with defects on either side of the tolerance's own size
        const double norm = std::sqrt(1.0 + 1e-4 * (2.0 * uni(rng) - 1.0));
        double na = 0.0, nb = 0.0;
        for (int s = 0; s < S; ++s) {
          const double e = std::ldexp(1.0, -(int)(rng() % 3));
          double x = 1.0;
          if (kind == 1) x = e * 1.0039;                                    // next to the tie between two bf16 values: the largest m
          if (kind == 2) x = e * (1.0 + 0.0039 + 3e-5 * uni(rng));          // ... with any l
          if (kind == 3) x = e * (1.0 + uni(rng));
          if (kind == 4) x = 2.0 * uni(rng) - 1.0;
          if (kind == 5) x = s == trial % S ? 1.0 : 1e-3 * uni(rng);
          a[s] = (float)x;
          b[s] = (float)(kind == 4 ? 2.0 * uni(rng) - 1.0 : x);
          na += (double)a[s] * a[s];
          nb += (double)b[s] * b[s];
        }
        const bool kept = (kind == 1 || kind == 2) && trial % 2;            // half of them as they are, but for a power of two
        const double fa = kept ? std::ldexp(1.0, -(int)std::ceil(0.5 * std::log2(na))) : norm / std::sqrt(na);
        const double fb = kept ? fa : norm / std::sqrt(nb);
        for (int s = 0; s < S; ++s) {
          a[s] = (float)(a[s] * fa);
          b[s] = (float)(b[s] * fb);
        }
        const double want = exact(a, b);
        for (int cut = 0; cut < 2; ++cut) {
          const double off = std::fabs((double)as_the_kernel(a, b, cut) - want);
          used = std::max(used, off / margin);
          if (!(off <= margin) && ++failures <= 10)
            std::printf("FAIL: %d rows, kind %d, trial %d, cut %d: off by %.3g, margin %.3g\n", S, kind, trial, cut, off, margin);
        }
      }
  }
  // what is left must still answer for a basis that is orthonormal to fp32, and fp32 matrices are never answered for
  for (int S : {1, 2048, 8192})
    if (!(refresh_check_tolerance(1e-4f, S) > 4e-5f) || refresh_check_tolerance(1e-6f, S) > 0.0f) { ++failures; std::printf("FAIL: tolerance at %d rows\n", S); }
  std::printf("largest share of the margin: %.3f\n%d failure(s)\n", used, failures);
  return failures != 0;
}
