// Host program behind test_norm_factor_host.py: the sums of norm_factor_kernel (csrc/norm_factor.h), dealt to its waves and lanes as the kernel deals
// them, against a row added up as its order is defined.  Prints the numbers of partials at which a bit differs.
#include "../paper_2510_01336_amd/csrc/norm_factor.h"
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

static float defined(const std::vector<float>& p) {      // 64 chains, whole turns of four sums, then neighbours
  const int n = (int)p.size();
  float t[64];
  for (int l = 0; l < 64; ++l) {
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    int i = l;
    for (; i + 192 < n; i += 256)
      for (int j = 0; j < 4; ++j) s[j] += p[i + 64 * j];
    for (; i < n; i += 64) s[0] += p[i];
    t[l] = (s[0] + s[1]) + (s[2] + s[3]);
  }
  for (int sh = 1; sh < 64; sh <<= 1) {                  // (both sides of a butterfly hold the same sum)
    float o[64];
    for (int l = 0; l < 64; ++l) o[l] = t[l] + t[l ^ sh];
    memcpy(t, o, sizeof(t));
  }
  return t[0];
}

static float dealt(const std::vector<float>& p) {
  const int n = (int)p.size();
  float wave_sum[16];
  for (int w = 0; w < 16; ++w) {
    float half[2];
    for (int h = 0; h < 2; ++h) {
      float s[2][4] = {};
      for (int i0 = 0; i0 < n; i0 += 256)
        for (int c = 0; c < 2; ++c) {
          float x[4];
          for (int j = 0; j < 4; ++j) x[j] = i0 + 4 * w + 2 * h + c + 64 * j < n ? p[i0 + 4 * w + 2 * h + c + 64 * j] : NAN;      // must not be added
          norm_chain_add(s[c], x, i0 + 4 * w + 2 * h + c, n);
        }
      half[h] = norm_chain_sum(s[0]) + norm_chain_sum(s[1]);
    }
    wave_sum[w] = half[0] + half[1];
  }
  return norm_tree(wave_sum);
}

int main() {
  std::mt19937 rng(5);
  std::lognormal_distribution<float> d(0.f, 3.f);
  int bad = 0;
  for (int n = 1; n <= 1100; ++n)
    for (int rep = 0; rep < 8; ++rep) {
      std::vector<float> p(n);
      for (float& x : p) x = rep == 7 ? 0.f : d(rng);
      const float a = defined(p), b = dealt(p);
      if (memcmp(&a, &b, sizeof(a)) && ++bad <= 20) printf("%d partials: %a, defined %a\n", n, b, a);
    }
  return bad != 0;
}
