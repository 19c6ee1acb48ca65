// sl_force.hip -- force kernels of the spin-lattice step on gfx950:
//   * k_eam_density: first pass of the embedded-atom terms;
//   * k_force:       pair + magneto-mechanical force (Eq. p_advance), fused
//                    with the velocity-Verlet half kicks and the drift into
//                    the other position buffer, energies on sampled steps
//                    and the per-block terms of the rebuild predictor;
//   * k_pred_reduce: one block joining those terms and handing them to the
//                    host.
#include "sl_step.h"

namespace sl {

// Densities: one workgroup on 64 atoms, every wavefront a quarter of the rows'
// rounds. Bound by the chain list entry, position, sum; with one wavefront per 64 atoms
// 128 000 atoms are two wavefronts per SIMD. Microseconds per step with one and four:
// 8192 atoms 59 and 56, 65 536 77 and 74, 128 000 87.5 and 85.5, 432 000 179 and 177
// (FP32 146.5 and 144.7).
constexpr int kDensityWaves = kBlock / 64;
template <typename real>
__global__ __launch_bounds__(kBlock) void k_eam_density(SysView<real> S, PotConst P) {
  __shared__ real part[kDensityWaves - 1][64];
  const int w = wave_id(), lane = threadIdx.x & 63;
  const int i = xcd_tile(blockIdx.x, gridDim.x) * 64 + lane;
  real rho = i < S.n ? eam_density_sum<real, kDensityWaves>(S, P, i, w) : (real)0;
  if (w > 0) part[w - 1][lane] = rho;
  __syncthreads();
  if (w > 0 || i >= S.n) return;
#pragma unroll
  for (int q = 0; q < kDensityWaves - 1; ++q) rho += part[q][lane];
  eam_density_store<real>(S, P, i, rho);
}

template <typename real>
void launch_eam_density(const SysView<real> &S, const PotConst &P, hipStream_t st) {
  if (S.n > 0 && P.eam_on && S.eam)
    hipLaunchKernelGGL((k_eam_density<real>), dim3((S.n + 63) / 64), dim3(kBlock), 0, st, S, P);
}
template void launch_eam_density<double>(const SysView<double> &, const PotConst &, hipStream_t);
template void launch_eam_density<float>(const SysView<float> &, const PotConst &, hipStream_t);


template <typename real, int MODE, int WAVES, int MLP>
__global__ __launch_bounds__(team_block(WAVES), kForceWaves) void k_force(SysView<real> S, PotConst P, ForceArgs A) {
  constexpr int kWv = team_block(WAVES) / 64, kAtoms = team_atoms(WAVES);
  __shared__ double red[kWv][8];
  __shared__ double redm[kWv][3];
  __shared__ ForceTeam<real, WAVES> team[WAVES > 1 ? kWv / WAVES : 1];
  // With a tile table (A.tiles) block b takes the atom range the host gave
  // it: XCD b % 8 holds the same spatial slab of every colour class, so its
  // L2 serves the neighbour gathers of all classes of that slab. Without
  // one, tiles are taken from the end of the atom order first: the last
  // colour classes may hold a few atoms scattered over the whole box
  // (repairs), whose gathers miss the caches; starting them first hides
  // their latency behind the bulk instead of leaving them as the tail.
  const int t = wave_id() / WAVES, w = wave_id() % WAVES;
  const int a = 64 * t + (int)(threadIdx.x & 63);  // atom of the block
  int tile, i;
  bool valid;
  if (A.tiles) {
    const int2 rg = A.tiles[blockIdx.x];
    tile = blockIdx.x;
    i = rg.x + a;
    valid = i < rg.y;
  } else {
    tile = gridDim.x - 1 - xcd_tile(blockIdx.x, gridDim.x);
    i = tile * kAtoms + a;
    valid = i < S.n;
  }
  double e[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  double dm = 0.0, vm = 0.0, wm = kInf;
  force_atom<real, MODE, WAVES, MLP>(S, P, A, i, valid, w, team + t, e, dm, vm, wm);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (MODE & kModeEnergy) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const double x = wave_sum(e[c]);
      if (lane == 0) red[wv][c] = x;
    }
  }
  if (MODE & (kModeFinal | kModeNext)) {
    const double xd = wave_max(dm), xv = wave_max(vm), xw = wave_min(wm);
    if (lane == 0) { redm[wv][0] = xd; redm[wv][1] = xv; redm[wv][2] = xw; }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (MODE & kModeEnergy) {
      for (int c = 0; c < 8; ++c) {
        double x = 0.0;
        for (int q = 0; q < kWv; ++q) x += red[q][c];
        A.partial[(size_t)tile * 8 + c] = x;
      }
    }
    // Predictor terms go out as plain per-block stores; k_pred_reduce joins
    // them. (Device-scope atomics on three shared words, plus a completion
    // counter, cost ~50 us per launch at 1688 blocks: they serialise across
    // the XCDs.)
    if (MODE & (kModeFinal | kModeNext)) {
      double xd = 0.0, xv = 0.0, xw = kInf;
      for (int q = 0; q < kWv; ++q) {
        xd = fmax(xd, redm[q][0]);
        xv = fmax(xv, redm[q][1]);
        xw = fmin(xw, redm[q][2]);
      }
      A.pred[(size_t)tile * 3 + 0] = xd;
      A.pred[(size_t)tile * 3 + 1] = xv;
      A.pred[(size_t)tile * 3 + 2] = xw;
    }
  }
}

// Joins the per-block predictor terms of one force launch (max, max, min:
// exact in any order) and writes them, with the sticky error word, to the
// pinned host slot; the written marker goes last.
__global__ __launch_bounds__(kBlock) void k_pred_reduce(const double *pred, int nb, int *err,
                                                        double *host_out, double mark) {
  __shared__ double s[3][kBlock / 64];
  double a = 0.0, b = 0.0, c = kInf;
  for (int k = threadIdx.x; k < nb; k += kBlock) {
    a = fmax(a, pred[(size_t)k * 3 + 0]);
    b = fmax(b, pred[(size_t)k * 3 + 1]);
    c = fmin(c, pred[(size_t)k * 3 + 2]);
  }
  a = wave_max(a);
  b = wave_max(b);
  c = wave_min(c);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) { s[0][wv] = a; s[1][wv] = b; s[2][wv] = c; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) {
      a = fmax(a, s[0][w]);
      b = fmax(b, s[1][w]);
      c = fmin(c, s[2][w]);
    }
    const int e = atomicOr(err, 0);
    host_out[0] = a;
    host_out[1] = b;
    host_out[2] = (double)e;
    host_out[4] = c;
    __threadfence_system();
    host_out[3] = mark;  // written marker
  }
}

void launch_pred_reduce(const double *pred, int nb, int *err, double *host_out, double mark,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_pred_reduce, dim3(1), dim3(kBlock), 0, st, pred, nb, err, host_out, mark);
}


template <typename real, int WAVES, int MLP>
static void force_lanes2(const SysView<real> &S, const PotConst &P, const ForceArgs &A,
                         hipStream_t st) {
  const int nb = A.tiles ? A.ntiles : force_blocks(S.n, WAVES);
  switch (A.mode) {
#define SL_FORCE_CASE(m) \
  case m: hipLaunchKernelGGL((k_force<real, m, WAVES, MLP>), dim3(nb), dim3(team_block(WAVES)), 0, st, S, P, A); break;
    SL_FORCE_CASE(1) SL_FORCE_CASE(2) SL_FORCE_CASE(3) SL_FORCE_CASE(4)
    SL_FORCE_CASE(5) SL_FORCE_CASE(6) SL_FORCE_CASE(7)
#undef SL_FORCE_CASE
    default: break;
  }
}

template <typename real, int WAVES>
static void force_lanes(const SysView<real> &S, const PotConst &P, const ForceArgs &A,
                        hipStream_t st) {
  if (P.soc_on && P.eam_on) force_lanes2<real, WAVES, 12>(S, P, A, st);
  else if (P.eam_on) force_lanes2<real, WAVES, 8>(S, P, A, st);
  else if (P.soc_on) force_lanes2<real, WAVES, 4>(S, P, A, st);
  else if (sizeof(real) == 4 && S.spl.t) force_lanes2<real, WAVES, (sizeof(real) == 4 ? 2 : 0)>(S, P, A, st);
  else if (sizeof(real) == 4 && S.tab) force_lanes2<real, WAVES, (sizeof(real) == 4 ? 1 : 0)>(S, P, A, st);
  else force_lanes2<real, WAVES, 0>(S, P, A, st);
}

// Pair pass of the split force: the spin-independent terms of every atom
// into A.fp (MODE is 0 or kModeEnergy: with it the pair energy is stored
// too). No reductions, kicks or predictor: the spin pass does those.
template <typename real, int MODE, int WAVES, int MLP>
__global__ __launch_bounds__(kBlock, kForceWaves) void k_pair(SysView<real> S, PotConst P, ForceArgs A) {
  __shared__ ForceTeam<real, WAVES> team[WAVES > 1 ? kBlock / 64 / WAVES : 1];
  const int tile = gridDim.x - 1 - xcd_tile(blockIdx.x, gridDim.x);
  const int t = wave_id() / WAVES, w = wave_id() % WAVES;
  const int i = tile * team_atoms(WAVES) + 64 * t + (int)(threadIdx.x & 63);
  double e[8];
  double dm = 0.0, vm = 0.0, wm = kInf;
  force_atom<real, MODE, WAVES, MLP | 16>(S, P, A, i, i < S.n, w, team + t, e, dm, vm, wm);
}

template <typename real, int WAVES, int MLP>
static void pair_lanes2(const SysView<real> &S, const PotConst &P, const ForceArgs &A,
                        bool energy, hipStream_t st) {
  const int nb = force_blocks(S.n, WAVES);
  if (energy)
    hipLaunchKernelGGL((k_pair<real, kModeEnergy, WAVES, MLP>), dim3(nb), dim3(kBlock), 0, st, S, P, A);
  else
    hipLaunchKernelGGL((k_pair<real, 0, WAVES, MLP>), dim3(nb), dim3(kBlock), 0, st, S, P, A);
}

template <typename real>
void launch_pair(const SysView<real> &S, const PotConst &P, const ForceArgs &A, int lanes,
                 bool energy, hipStream_t st) {
  if (S.n <= 0) return;
  if (lanes == 2) {
    if (P.eam_on) pair_lanes2<real, 2, 8>(S, P, A, energy, st);
    else pair_lanes2<real, 2, 0>(S, P, A, energy, st);
  } else {
    if (P.eam_on) pair_lanes2<real, 1, 8>(S, P, A, energy, st);
    else pair_lanes2<real, 1, 0>(S, P, A, energy, st);
  }
}
template void launch_pair<double>(const SysView<double> &, const PotConst &, const ForceArgs &, int,
                                  bool, hipStream_t);
template void launch_pair<float>(const SysView<float> &, const PotConst &, const ForceArgs &, int,
                                 bool, hipStream_t);

// Spin pass of the split force (the pair pass must have filled A.fp).
template <typename real>
void launch_force_spin(const SysView<real> &S, const PotConst &P, const ForceArgs &A, int lanes,
                       hipStream_t st) {
  if (S.n <= 0) return;
  if (lanes == 2) {
    if (P.soc_on) force_lanes2<real, 2, 4 | 32>(S, P, A, st);
    else force_lanes2<real, 2, 32>(S, P, A, st);
  } else {
    if (P.soc_on) force_lanes2<real, 1, 4 | 32>(S, P, A, st);
    else force_lanes2<real, 1, 32>(S, P, A, st);
  }
}
template void launch_force_spin<double>(const SysView<double> &, const PotConst &,
                                        const ForceArgs &, int, hipStream_t);
template void launch_force_spin<float>(const SysView<float> &, const PotConst &, const ForceArgs &,
                                       int, hipStream_t);

// Blocks needed by a force launch (rows of the partial-sum buffer).
int force_block_atoms(int waves) { return team_atoms(waves); }
int force_blocks(int n, int waves) { return (n + team_atoms(waves) - 1) / team_atoms(waves); }

template <typename real>
void launch_force(const SysView<real> &S, const PotConst &P, const ForceArgs &A, int lanes,
                  hipStream_t st) {
  if (S.n <= 0) return;
  switch (lanes) {
    case 1: force_lanes<real, 1>(S, P, A, st); break;
    case 2: force_lanes<real, 2>(S, P, A, st); break;
    case 8: force_lanes<real, 8>(S, P, A, st); break;
    default: force_lanes<real, 4>(S, P, A, st); break;
  }
}


template void launch_force<double>(const SysView<double> &, const PotConst &, const ForceArgs &,
                                   int, hipStream_t);
template void launch_force<float>(const SysView<float> &, const PotConst &, const ForceArgs &, int,
                                  hipStream_t);

}  // namespace sl
