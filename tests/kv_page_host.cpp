// Host program behind test_kv_page_host.py: enumerates the offsets of a KV page for every head size a model may have and
// prints those whose positions and dimensions do not each own one element inside the slab.
#include "../paper_2510_01336_amd/csrc/common.h"
#include <cstdio>

int main() {
  int bad = 0;
  for (int D = 2; D <= 256; D += 2) {
    const size_t slab = kv_slab(0, 0, 1, 1, 2, D), v0 = (size_t)EE_PAGE * kv_page_dim(D);
    std::vector<int> owner(slab, 0);
    int wrong = 0;
    for (int pos = 0; pos < EE_PAGE; ++pos)
      for (int d = 0; d < D; ++d)
        for (size_t o : {(size_t)k_page_off(pos, d, D), v0 + v_page_off(pos, d)}) {
          if (o >= slab || owner[o]++) ++wrong;
        }
    // the fp32 attention reads eight dimensions of K, eight positions of V at once
    for (int pos = 0; pos < EE_PAGE; ++pos)
      for (int d = 0; d < D; ++d) {
        if (d % 8 == 0 && k_page_off(pos, d, D) % 8) ++wrong;
        if (pos % 8 == 0 && v_page_off(pos, d) % 8) ++wrong;
      }
    if (wrong) { printf("head_dim %d: %d\n", D, wrong); ++bad; }
  }
  return bad != 0;
}
