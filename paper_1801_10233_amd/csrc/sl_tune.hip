// sl_tune.hip -- the autotuner of a single system: times launch shapes on
// scratch copies and keeps the fastest (JSON-lines cache optional).
#include "sl_host.h"

// ============================================================================
// Autotuner: times launch shapes on scratch copies and keeps the fastest.
namespace sl {

// State of S in user order, masses included.
int user_state(sl_system *S, std::vector<double> &r, std::vector<double> &v,
               std::vector<double> &sp, std::vector<double> &m) {
  const int n = S->n;
  r.resize(3 * (size_t)n);
  v.resize(3 * (size_t)n);
  sp.resize(3 * (size_t)n);
  m.resize(n);
  CHK(sl_get_state(S, r.data(), v.data(), sp.data(), SL_HOST));
  std::vector<double> mi(n);
  std::vector<int> id(n);
  Atoms &A = S->a[S->cur];
  HIPCHK(S, hipMemcpy(mi.data(), A.mass, sizeof(double) * n, hipMemcpyDeviceToHost));
  HIPCHK(S, hipMemcpy(id.data(), A.id, sizeof(int) * n, hipMemcpyDeviceToHost));
  for (int i = 0; i < n; ++i) m[id[i]] = mi[i];
  if (S->prec == SL_FP32)  // FP32 spins are unit to FP32 rounding only
    for (int i = 0; i < n; ++i) {
      double *q = &sp[3 * (size_t)i];
      const double inv = 1.0 / std::sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
      q[0] *= inv; q[1] *= inv; q[2] *= inv;
    }
  return SL_OK;
}

// Scratch copy of S (parameters, interactions, learned potential, user
// list, state and step counter) on its own stream.
int clone_system(sl_system *S, sl_system **out) {
  *out = nullptr;
  CHK(sl_synchronize(S));
  sl_params p = S->prm;
  p.stream = nullptr;
  p.skin = S->skin;
  p.max_nbr = S->max_nbr;
  p.max_spin_nbr = S->max_spin;
  sl_system *C = nullptr;
  int rc = sl_create(&p, &C);
  if (rc) return fail(S, rc, std::string("autotune copy: ") + sl_last_error(nullptr));
  auto bail = [&](int code) {
    const std::string e = C->last_err;
    sl_destroy(C);
    return fail(S, code, "autotune copy: " + e);
  };
  if ((rc = sl_set_potential(C, &S->pot))) return bail(rc);
  std::vector<double> r, v, sp, m;
  CHK(user_state(S, r, v, sp, m));
  if ((rc = sl_set_state(C, r.data(), v.data(), sp.data(), m.data(), SL_HOST))) return bail(rc);
  if (S->user_list) {
    const int n = S->n;
    std::vector<int> ns(n), na(n);
    const int64_t tot = sl_get_neighbor_list(S, ns.data(), na.data(), nullptr, 0);
    if (tot < 0) return bail((int)tot);
    std::vector<int> idx(std::max<int64_t>(tot, 1)), off(n + 1, 0);
    const int64_t t2 = sl_get_neighbor_list(S, ns.data(), na.data(), idx.data(), tot);
    if (t2 < 0) return bail((int)t2);
    for (int i = 0; i < n; ++i) off[i + 1] = off[i] + na[i];
    if ((rc = sl_set_neighbor_list(C, off.data(), idx.data(), SL_HOST))) return bail(rc);
  }
  if (S->mlp && (rc = sl_set_mlp(C, S->mlp))) return bail(rc);
  if (S->mlp && (rc = sl_set_mlp_mode(C, S->mlp_mode))) return bail(rc);
  if ((rc = sl_set_ordering(C, S->ordering, S->sgrid))) return bail(rc);
  if ((rc = sl_set_row_order(C, S->row_q))) return bail(rc);
  if ((rc = sl_set_step(C, S->step))) return bail(rc);
  // and the colour classes, as a repair at these positions leaves them: a run from a
  // perfect lattice keeps few large classes, a fresh colouring of its displaced atoms
  // has more and smaller ones, for which other shapes are the fastest (432 000 atoms
  // after 60 steps: 4 classes and 11)
  if (S->K > 0 && S->have_colour) {
    if ((rc = ensure_ready(C))) return bail(rc);
    const int n = S->n;
    std::vector<int> cu(n), ci(n), id(n);
    if ((rc = sl_get_coloring(S, cu.data(), nullptr))) return bail(rc);
    Atoms &A = C->a[C->cur];
    if (hipMemcpy(id.data(), A.id, sizeof(int) * n, hipMemcpyDeviceToHost) != hipSuccess) return bail(SL_E_HIP);
    for (int i = 0; i < n; ++i) ci[i] = cu[id[i]];
    if (hipMemcpy(A.colour, ci.data(), sizeof(int) * n, hipMemcpyHostToDevice) != hipSuccess) return bail(SL_E_HIP);
    C->Kbase = S->Kbase;
    if ((rc = rebuild(C))) return bail(rc);
  }
  *out = C;
  return SL_OK;
}

// Optional cache of tuned shapes: one JSON object per line in the file named
// by SL_TUNE_CACHE, keyed by the device and the workload's shape.
std::string tune_key(const std::string &what) {
  hipDeviceProp_t prop;
  int dev = 0;
  std::string arch = "unknown";
  if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
    arch = prop.gcnArchName;
  return arch + " " + what;
}

bool cache_lookup(const std::string &key, int vals[4]) {
  const char *path = std::getenv("SL_TUNE_CACHE");
  if (!path) return false;
  FILE *f = std::fopen(path, "r");
  if (!f) return false;
  char line[1024];
  bool found = false;
  const std::string want = "{\"key\": \"" + key + "\"";
  while (std::fgets(line, sizeof(line), f)) {
    if (std::strncmp(line, want.c_str(), want.size()) != 0) continue;
    const char *q = std::strstr(line, "\"vals\": [");
    if (q && std::sscanf(q, "\"vals\": [%d, %d, %d, %d]", &vals[0], &vals[1], &vals[2], &vals[3]) == 4)
      found = true;
  }
  std::fclose(f);
  return found;
}

void cache_store(const std::string &key, const int vals[4]) {
  const char *path = std::getenv("SL_TUNE_CACHE");
  if (!path) return;
  FILE *f = std::fopen(path, "a");
  if (!f) return;
  std::fprintf(f, "{\"key\": \"%s\", \"vals\": [%d, %d, %d, %d]}\n", key.c_str(), vals[0], vals[1],
               vals[2], vals[3]);
  std::fclose(f);
}

}  // namespace sl

extern "C" {

int sl_autotune(sl_system *S, int steps, double dt, sl_tuning *chosen) {
  if (!S || steps < 1 || !std::isfinite(dt) || dt == 0.0) return fail(S, SL_E_ARG, "bad autotune arguments");
  CHK(ensure_ready(S));
  // ("lanes=set": lines from when a force-lane count was only the least that ran lack it
  // and are not found)
  const std::string key = tune_key(
      "system lanes=set n=" + std::to_string(S->n) + " prec=" + std::to_string(S->prec) +
      " frozen=" + std::to_string(S->prm.frozen) + " langevin=" + std::to_string(S->pc.langevin) +
      " aniso=" + std::to_string(S->pc.aniso_on) + " mlp=" + std::to_string(S->mlp ? 1 : 0) +
      " K=" + std::to_string(S->K));
  int v[4];
  if (!cache_lookup(key, v)) {
    sl_system *C = nullptr;
    CHK(clone_system(S, &C));
    // Every candidate (spin lanes, force lanes, J cache) runs a window of
    // `steps` steps on the clone, timed with events on its stream: the whole
    // step counts, so the cache's own kernel and its effect on the other
    // kernels (it shares the caches with them) are part of the comparison.
    // A window with a list rebuild in it is run again; four rounds over
    // all candidates, the best window of each counts.
    const std::vector<sl_tuning> trial = tune_candidates(S);
    const int ntrial = (int)trial.size();
    std::vector<double> best(ntrial, 1e300);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = SL_OK;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = SL_E_HIP;
    // sustained load first: the device's clocks and caches then are those of
    // a long run, not of a device that has just been idle
    if (rc == SL_OK) rc = sl_step(C, 6 * steps, dt);
    // the order of the candidates rotates from round to round, so no shape
    // always follows the same other one
    for (int pass = 0; pass < 4 && rc == SL_OK; ++pass)
      for (int q = 0; q < ntrial && rc == SL_OK; ++q) {
        const int t = (q + 3 * pass) % ntrial;
        if ((rc = sl_set_tuning(C, &trial[t]))) break;
        if ((rc = sl_step(C, 3, dt))) break;
        for (int attempt = 0; attempt < 3 && rc == SL_OK; ++attempt) {
          const int64_t rb0 = C->rebuilds;
          if (hipEventRecord(e0, C->st) != hipSuccess) { rc = SL_E_HIP; break; }
          if ((rc = sl_step(C, steps, dt))) break;
          if (hipEventRecord(e1, C->st) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
            rc = SL_E_HIP;
            break;
          }
          float ms = 0.f;
          if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { rc = SL_E_HIP; break; }
          if (C->rebuilds != rb0) continue;  // a rebuild in the window: run it again
          best[t] = std::min(best[t], (double)ms / steps);
          break;
        }
      }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    const std::string err = rc ? C->last_err : std::string();
    sl_destroy(C);
    if (rc) return fail(S, rc, "autotune trial: " + err);
    int bt = 0;
    for (int t = 1; t < ntrial; ++t)
      if (best[t] < best[bt]) bt = t;
    v[0] = trial[bt].spin_lanes;
    v[1] = trial[bt].force_lanes;
    v[2] = S->small_class;
    v[3] = trial[bt].jcache;
    cache_store(key, v);
  }
  sl_tuning t{v[0], v[1], v[2], v[3], S->overlap};
  CHK(sl_set_tuning(S, &t));
  return chosen ? sl_get_tuning(S, chosen) : SL_OK;
}

}  // extern "C"
