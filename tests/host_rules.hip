// Rules by which the host code picks kernels and launch shapes, printed as
// "name value" lines (no device is used).
#include <cstdio>

#include "../paper_1801_10233_amd/csrc/sl_host.h"

using namespace sl;

template <typename real>
static void variants(const char *tag) {
  real c[1];
  SysView<real> with{}, without{};
  PotConst P{};
  with.jc = c;
  std::printf("%s_cache_at_both %d\n", tag, spin_variant(with, P, &with));
  std::printf("%s_cache_at_first %d\n", tag, spin_variant(with, P, &without));
  std::printf("%s_cache_at_second %d\n", tag, spin_variant(without, P, &with));
  std::printf("%s_cache_single %d\n", tag, spin_variant<real>(with, P, nullptr));
  float4 t[1];
  with.spl.t = without.spl.t = t;
  std::printf("%s_spline_cache_at_first %d\n", tag, spin_variant(with, P, &without));
}

int main() {
  variants<double>("fp64");
  variants<float>("fp32");
  for (long nbucket : {1L, 5L, 16384L, 1L << 26, 1L << 30})
    std::printf("sort_threads_%ld %ld\n", nbucket, (long)bucket_sort_blocks((int)nbucket) * kBlock);
  for (int rows : {1, 5, 6, 63, 80, 640, 641, 400000}) {
    const int slots = slots_per_group(rows, 5);
    std::printf("slots_%d %d\n", rows, slots);
    std::printf("groups_%d %d\n", rows, (rows + slots - 1) / slots);
  }
  return 0;
}
