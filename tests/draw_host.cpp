// Host program behind test_draw_host.py: the inverse-CDF draw of kernels_sample.hip in plain loops -- the same sums in the same
// order as a workgroup of sixteen 64-lane waves forms them (butterfly sums, shuffle-up scans), the decisions from csrc/draw.h.
// Usage: draw_host VOCAB ROWS DRAWS SEED; prints draws, tokens of weight zero, tokens whose CDF interval misses the target by
// more than 8e-6 of the total.
#include "../paper_2510_01336_amd/csrc/draw.h"
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <random>
#include <vector>

static void scan(float v[64]) {                       // wave_scan
  for (int s = 1; s < 64; s <<= 1) {
    float o[64];
    for (int l = 0; l < 64; ++l) o[l] = l >= s ? v[l - s] : 0.f;
    for (int l = s; l < 64; ++l) v[l] += o[l];
  }
}
static float sum(float v[64]) {                       // wave_sum
  for (int s = 1; s < 64; s <<= 1) {
    float o[64];
    for (int l = 0; l < 64; ++l) o[l] = v[l ^ s];
    for (int l = 0; l < 64; ++l) v[l] += o[l];
  }
  return v[0];
}

struct Row {
  std::vector<float> w;
  int vocab, R, per;
  std::vector<float> group, incl, inc;                // [16][64], [16][64], [chunk][64]: scans of the lanes' four-token sums
  float tot[16], total;
  int end;
  float4 four(int i) const {
    auto at = [&](int k) { return k < vocab ? w[k] : 0.f; };
    return make_float4(at(i), at(i + 1), at(i + 2), at(i + 3));
  }
  explicit Row(std::vector<float> x) : w(std::move(x)) {
    vocab = (int)w.size();
    R = (vocab + 4095) / 4096 * 256; per = (R / 256 + 63) / 64;
    group.assign(16 * 64, 0.f); incl = group; inc.assign((size_t)16 * (R / 256) * 64, 0.f);
    end = -1;
    for (int i = 0; i < vocab; ++i) if (w[i] > 0.f) end = i;
    total = 0.f;
    for (int v = 0; v < 16; ++v) {
      for (int c = 0; c < R / 256; ++c) {
        float b[64], *n = &inc[((size_t)v * (R / 256) + c) * 64];
        for (int l = 0; l < 64; ++l) {
          const float4 x4 = four(v * R + c * 256 + 4 * l);
          b[l] = (x4.x + x4.y) + (x4.z + x4.w);
          n[l] = ((x4.x + x4.y) + x4.z) + x4.w;
        }
        group[v * 64 + c / per] += sum(b);
        scan(n);
      }
      std::copy(&group[v * 64], &group[v * 64] + 64, &incl[v * 64]);
      scan(&incl[v * 64]);
      tot[v] = incl[v * 64 + 63];
      total += tot[v];
    }
  }
  // the wave of a target and the sum of the waves before it
  int wave(float target, float& pre) const {
    pre = 0.f;
    for (int k = 0; k < 16; ++k) {
      if (pre + tot[k] > target) return k;
      pre += tot[k];
    }
    return -1;
  }
  int draw(float u) const {
    const float target = u * total;
    float pre;
    const int h = wave(target, pre);
    if (h < 0) return end;
    int gl = -1, held = -1;
    for (int l = 63; l >= 0; --l) {
      if (draw_admits_group(pre + incl[h * 64 + l], group[h * 64 + l], target)) gl = l;
      if (held < 0 && group[h * 64 + l] > 0.f) held = l;
    }
    if (gl < 0) gl = held;
    float run = pre + (gl ? incl[h * 64 + gl - 1] : 0.f);
    int tok = -1, seen = -1;
    const int i1 = std::min(vocab, (h + 1) * R);
    for (int c = 0; c < per && tok < 0; ++c) {
      const int chunk = gl * per + c, i0 = h * R + chunk * 256;
      if (i0 >= i1) break;
      const float* n = &inc[((size_t)h * (R / 256) + chunk) * 64];
      for (int l = 0; l < 64; ++l) {
        const float4 x = four(i0 + 4 * l);
        const float s3 = ((x.x + x.y) + x.z) + x.w;
        const int k = draw_among_four(run + (n[l] - s3), x, target), mine = draw_last_of_four(x);
        if (k < 4 && tok < 0) tok = i0 + 4 * l + k;
        if (mine >= 0) seen = i0 + 4 * l + mine;
      }
      run += n[63];
    }
    return tok >= 0 ? tok : (seen >= 0 ? seen : end);
  }
};

int main(int argc, char** argv) {
  if (argc < 5) return 2;
  const int vocab = atoi(argv[1]), rows = atoi(argv[2]), draws = atoi(argv[3]);
  std::mt19937 rng(atoi(argv[4]));
  std::uniform_real_distribution<float> uni(0.f, 1.f);
  std::normal_distribution<float> gauss;
  long n = 0, zero = 0, far_off = 0;
  for (int r = 0; r < rows; ++r) {
    // residual max(0, p - q) of two softmax rows; every third row keeps few tokens only (empty groups and waves)
    std::vector<double> e[2];
    double s[2] = {0., 0.};
    const float spread = 0.3f + 3.f * uni(rng);
    for (int t = 0; t < 2; ++t) {
      e[t].resize(vocab);
      for (auto& x : e[t]) s[t] += x = std::exp((double)(spread * gauss(rng)));
    }
    std::vector<float> w(vocab);
    const float keep = r % 3 == 2 ? 30.f / vocab : 2.f;
    for (int i = 0; i < vocab; ++i) {
      const float p = (float)(e[0][i] / s[0]), q = (float)(e[1][i] / s[1]);
      w[i] = uni(rng) < keep ? fmaxf(0.f, p - q) : 0.f;
    }
    const Row row(w);
    if (!(row.total > 0.f)) continue;
    std::vector<double> cdf(vocab + 1, 0.);
    for (int i = 0; i < vocab; ++i) cdf[i + 1] = cdf[i] + (double)w[i];
    for (int k = 0; k < draws; ++k) {
      // every other number lands on the edge of a lane's four tokens or of a group of chunks, a few ulp either way
      float u = uni(rng);
      if (k & 1) {
        const int edge = k & 2 ? 256 * row.per : 4, i = (int)(uni(rng) * (vocab / edge)) * edge;
        u = (float)(cdf[i] / cdf[vocab]);
        for (int j = (int)(rng() % 17) - 8; j != 0; j -= j > 0 ? 1 : -1) u = std::nextafterf(u, j > 0 ? 1.f : 0.f);
        u = fminf(fmaxf(u, 0.f), 0.99999994f);
      }
      const int tok = row.draw(u);
      ++n;
      const double at = (double)u * cdf[vocab], tol = 8e-6 * cdf[vocab];
      if (tok < 0 || !(w[tok] > 0.f)) ++zero;
      if (tok < 0 || cdf[tok] - tol > at || cdf[tok + 1] + tol < at) ++far_off;
    }
  }
  printf("%ld %ld %ld\n", n, zero, far_off);
  return 0;
}
