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

// Autotuner candidates of a system of K equal classes: their number, whether the first
// is the default, and the number of distinct launch shapes among them.
static void candidates(const char *tag, int prec, int n, int K, bool frozen, bool soc) {
  sl_system S;
  S.prec = prec;
  S.n = n;
  S.K = K;
  S.jcache = prec == SL_FP32 ? 1 : -1;
  S.prm.frozen = frozen;
  S.pc.soc_on = soc;
  S.prof = true;  // (timing the caller's launches does not narrow the choice)
  for (int c = 0; c <= K; ++c) S.class_off.push_back((int)((long)n * c / K));
  const std::vector<sl_tuning> t = tune_candidates(&S);
  std::vector<std::vector<int>> shapes;
  int distinct = 0, cached = 0;
  for (const sl_tuning &x : t) {
    sl_system D = S;
    D.prof = false;
    apply_tuning(&D, x);
    const std::vector<int> v = launch_shape(&D);
    distinct += std::find(shapes.begin(), shapes.end(), v) == shapes.end();
    cached += v.back();
    shapes.push_back(v);
  }
  std::printf("%s_count %d\n%s_distinct %d\n%s_cached %d\n", tag, (int)t.size(), tag, distinct, tag, cached);
  std::printf("%s_default_first %d\n", tag, t[0].spin_lanes == 0 && t[0].force_lanes == 0 && t[0].jcache == 0);
  std::printf("%s_default_one_workgroup %d\n", tag, shapes[0][0] == 0);
}

int main() {
  candidates("small", SL_FP64, 1024, 4, false, false);
  candidates("middle", SL_FP64, 24334, 10, false, false);
  candidates("middle_fp32", SL_FP32, 24334, 10, false, false);
  candidates("large", SL_FP64, 432000, 4, false, false);
  candidates("frozen", SL_FP64, 65536, 4, true, false);
  candidates("soc", SL_FP64, 27648, 10, false, true);
  variants<double>("fp64");
  variants<float>("fp32");
  for (long nbucket : {1L, 5L, 16384L, 1L << 26, 1L << 30})
    std::printf("sort_threads_%ld %ld\n", nbucket, (long)bucket_sort_blocks((int)nbucket) * kBlock);
  for (int prec : {SL_FP64, SL_FP32}) {
    sl_system S;
    S.prec = prec;
    apply_tuning(&S, {0, 0, 0, 1, 0});
    std::printf("cache_%d_on %d\n", prec, jcache_on(&S));
    S.jc_failed = true;
    std::printf("cache_%d_failed %d\n", prec, jcache_on(&S));
    apply_tuning(&S, {0, 0, 0, 1, 0});
    std::printf("cache_%d_set_again %d\n", prec, jcache_on(&S));
  }
  for (int rows : {1, 5, 6, 63, 80, 640, 641, 400000}) {
    const int slots = slots_per_group(rows, 5);
    std::printf("slots_%d %d\n", rows, slots);
    std::printf("groups_%d %d\n", rows, (rows + slots - 1) / slots);
  }
  for (int prec : {SL_FP64, SL_FP32})
    for (int jc : {-1, 1})
      for (int m : {1, 3000, 3001, 70000, 70001, 108000}) {
        sl_system S;
        S.prec = prec;
        S.jcache = jc;
        S.jc_auto = false;
        std::printf("spin_lanes_%d_%d_%d %d\n", prec, jc, m, spin_lanes_for(&S, m));
      }
  for (int n : {1, 12000, 12001, 120000, 120001, 432000}) {
    sl_system S;
    S.n = n;
    std::printf("force_lanes_%d %d\n", n, force_lanes_for(&S));
    for (int lanes : {1, 2, 4, 8})
      for (int overlap : {-1, 1}) {
        apply_tuning(&S, {0, lanes, 0, 0, overlap});
        std::printf("force_lanes_%d_set_%d_%d %d\n", n, lanes, overlap, force_lanes_for(&S));
      }
    apply_tuning(&S, {0, 0, 0, 0, 1});
    std::printf("force_lanes_%d_split %d\n", n, force_lanes_for(&S));
  }
  return 0;
}
