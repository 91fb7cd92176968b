// split_rule.cpp -- asks the retrieval's rule for one wave per component
// (split_plan) about stores given on standard input, a line each:
//   dtype codec full0 full words_per_wave i0 k waves box
// and prints, per line, "0" or "1 i1 lds_bytes".
#include <cstdio>

#include "../../paper_2308_11759_amd/csrc/internal.hpp"

int main() {
  int dtype, codec, i0, k, box;
  unsigned long long full0, full, span, waves;
  while (std::scanf("%d %d %llu %llu %llu %d %d %llu %d", &dtype, &codec, &full0, &full, &span, &i0, &k, &waves, &box) == 9) {
    pmc_store s;
    s.f.dtype = dtype;
    s.codec = codec;
    s.n = k;
    s.max_span.assign(k, span);
    s.full.assign(k, full);
    s.full[0] = full0;
    pmc::SplitArgs sp{};
    int i1 = 0;
    if (pmc_host::split_plan(&s, i0, k, waves, box != 0, &i1, &sp)) std::printf("1 %d %u\n", i1, sp.lds_bytes);
    else std::printf("0\n");
  }
  return 0;
}
