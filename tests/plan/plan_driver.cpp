// plan_driver.cpp -- prints the plans of the library it is linked to, for the CPU tests.
// A line "n nsets n_leaf flags" of the input gives one of the output: the fields of the
// plan as "name value" pairs.  With the argument "walk" a line "n c_max" gives the walk's
// items of work.  No GPU is touched.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "tb_internal.h"

int main(int argc, char **argv) {
  if (argc > 1 && std::strcmp(argv[1], "walk") == 0) {
    long long n, c_max;
    while (std::scanf("%lld %lld", &n, &c_max) == 2) {
      const tb::WalkItems it = tb::walk_items(n, c_max);
      std::printf("part %d whole %d\n", (int)it.part, it.whole ? 1 : 0);
    }
    return 0;
  }
  int32_t shapes[3 * 64];
  int count = 0;
  if (tb_sort_configs(shapes, 64, &count) != TB_OK) return 1;
  long long n, nsets, n_leaf;
  unsigned long flags;
  while (std::scanf("%lld %lld %lld %lu", &n, &nsets, &n_leaf, &flags) == 4) {
    const int k = (int)((flags >> 8) & 0xffu);
    if (k >= count) return 1;
    const tb::SortConfig asked = {shapes[3 * k], shapes[3 * k + 1], shapes[3 * k + 2]};
    tb::Plan p;
    if (tb::make_plan(n, (int32_t)nsets, (int32_t)n_leaf, (uint32_t)flags, asked, &p) != TB_OK)
      return 1;
    std::printf("cell_tile %d cell_tiles %lld group_levels %d total %zu bits %d idx_bits %d "
                "key_passes %d low_passes %d skip_bits %d counted %u",
                p.cell_tile, (long long)p.cell_tiles, tb::group_levels(p), p.total, p.sort.bits,
                p.idx_bits, p.key_passes, p.low_passes, p.skip_bits, p.counted);
    std::printf(" low_packed %d", p.low_packed ? 1 : 0);
    for (int k = 0; k < p.low_passes; ++k) std::printf(" low%d %d", k, tb::low_shift(p, k));
    for (int k = 0; k <= p.key_passes; ++k) std::printf(" form%d %d", k, (int)p.form[k]);
    for (int k = 0; k < p.key_passes; ++k)
      std::printf(" built%d %d", k, tb::sort_pair_built(p.form[k], p.form[k + 1]) ? 1 : 0);
    std::printf("\n");
  }
  return 0;
}
