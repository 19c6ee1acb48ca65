// sl_dyn.hip -- spin kernels of the spin-lattice step on gfx950:
//   * k_spin_phase: one colour class of a spin sweep (Sec. 3 / Sec. 5.1);
//   * k_spin_tail:  a run of small classes in one workgroup;
//   * k_spin_lds:   the spin half-steps of a small system in one workgroup;
//   * k_jcache:     the optional exchange-coefficient cache;
//   * k_reduce8:    fixed-order second pass of the block partial sums.
#include "sl_step.h"

#ifndef SL_JC_CHUNK
#define SL_JC_CHUNK 5  // list slots per round of the exchange-cache kernel
                       // (3, 4 and 5 measured alike, 6, 7, 8 and 14 slower)
#endif

#include <climits>

#ifndef SL_JC_SPLIT
#define SL_JC_SPLIT 131072
#endif

namespace sl {

constexpr int kJcSplitAtoms = SL_JC_SPLIT;  // below: the row's slots split over grid.y

// (an argument block is written across the bus for each launch: no second view
// where it isn't read)
struct NoView {};
template <typename real, bool DUAL>
using SecondView = std::conditional_t<DUAL, SysView<real>, NoView>;

template <typename real, bool LANGEVIN, bool ANISO, int LANES, int MLP, bool DUAL>
__global__ __launch_bounds__((64 * TeamShape<LANES, LANGEVIN>::waves)) void k_spin_phase(
    const int *nbr, const void *p1, const void *p2, const void *p3, const void *p4, int begin, int end, int ld,
    int kcap, SysView<real> S, PotConst P, SpinPhaseArgs A, SecondView<real, DUAL> S2) {
  using T = TeamShape<LANES, LANGEVIN>;  // one workgroup per team
  __shared__ SpinTeam<real, T::waves> team[1];
  constexpr bool kCoeff = MLP == 1 || MLP == 3;
  // what the first loads need, in registers when the wavefront starts
  // (-amdgpu-kernarg-preload-count): the argument block itself is a trip to memory
  // (24 334 atoms, 31 spin launches per step: 201 us per step without, 189 with)
  S.nbr = nbr;
  if (kCoeff) {
    if (MLP == 3) S.jc = (const real *)p1;
    else S.tab = (const float4 *)p1;
    S.sx = (real *)p2;
    S.sy = (real *)p3;
    S.sz = (real *)p4;
  } else {
    S.rx = (const double *)p1;
    S.ry = (const double *)p2;
    S.rz = (const double *)p3;
    S.sx = (real *)p4;
  }
  S.ld = ld;
  S.kcap = kcap;
  const int nb = (end - begin + T::atoms - 1) / T::atoms;
  const int i = begin + xcd_tile(blockIdx.x, nb) * T::atoms + (int)(threadIdx.x & (T::atoms - 1));
  const SysView<real> *V2 = nullptr;
  if constexpr (DUAL) V2 = &S2;
  spin_update<real, LANGEVIN, ANISO, LANES, MLP, DUAL>(S, P, i, i < end, wave_id(), team, A.nrep, A.step, A.sub,
                                                       A.h, A.amp, A.seed, A.replica, A.rs2, V2,
                                                       !DUAL && A.keep != 0);
}

// A run of small classes (a few atoms each, e.g. the extra colours a repair
// adds) in one workgroup: the items are applied in order with a workgroup
// barrier between them, which keeps the class order of the sweep while
// paying one launch for the whole run. Teams of kTailLanes wavefronts whatever
// the launch shape of the large classes. Classes of more than the 128 atoms that
// such teams take in one pass (a set small_class) go on kTailWide wavefronts per 64
// atoms, in FP32 with ready coefficients also with twice the threads (from positions that
// is more than 128 registers), where fewer passes outweigh the longer ones (at most
// kTailWide successive updates draw their noise there). Microseconds per
// step with the bath, classes of 128 and up to 1024 atoms or so in one run: FP64
// 3456 atoms 437 on four wavefronts, 360 on two; FP32 362 and 276.
constexpr int kTailLanes = 4, kTailWide = 2;
template <typename real, int LANES, int MLP>
constexpr int kTailThreads =
    sizeof(real) == 4 && LANES == kTailWide && (MLP == 1 || MLP == 3) ? 1024 : kTailBlock;
template <int ATOMS>
struct TailSeq {
  const TailArgs &T;
  int item, base;
  __device__ bool more() const { return item < T.nitems; }
  __device__ int begin() const { return base; }
  __device__ int end() const { return T.item[item].end; }
  __device__ int nrep() const { return T.item[item].nrep; }
  __device__ int64_t step(int r) const { return T.item[item].step[r]; }
  __device__ int sub(int r) const { return T.item[item].sub[r]; }
  template <typename real> __device__ const float4 *tab(const SysView<real> &S) const { return S.tab; }
  template <typename real> __device__ const real *jc(const SysView<real> &S) const { return S.jc; }
  __device__ void advance() {
    base += ATOMS;
    if (base >= T.item[item].end && ++item < T.nitems) base = T.item[item].begin;
  }
  __device__ explicit TailSeq(const TailArgs &t) : T(t), item(0), base(t.item[0].begin) {}
  __device__ TailSeq(const TailSeq &o) = default;
  __device__ TailSeq &operator=(const TailSeq &o) {
    item = o.item;
    base = o.base;
    return *this;
  }
};
template <typename real, bool LANGEVIN, bool ANISO, int LANES, int MLP>
__global__ __launch_bounds__((kTailThreads<real, LANES, MLP>)) void k_spin_tail(SysView<real> S, PotConst P,
                                                          TailArgs T) {
  constexpr int kTeams = kTailThreads<real, LANES, MLP> / 64 / LANES;
  __shared__ SpinTeam<real, LANES> team[kTeams];
  if constexpr (MLP != 4) {
    spin_sequence<real, LANGEVIN, ANISO, LANES, kTeams, MLP>(TailSeq<64 * kTeams>(T), S, P, S.sx, S.sy, S.sz, team, T.h,
                                                                  T.amp, T.seed, T.replica, T.rs2);
  } else {
    const int t = wave_id() / LANES, w = wave_id() % LANES;
    for (int q = 0; q < T.nitems; ++q) {
      const TailItem &it = T.item[q];
      for (int base = it.begin; base < it.end; base += 64 * kTeams) {
        const int i = base + 64 * t + (int)(threadIdx.x & 63);
        spin_update<real, LANGEVIN, ANISO, LANES, MLP>(S, P, i, i < it.end, w, team + t, it.nrep,
                                                            it.step, it.sub, T.h, T.amp, T.seed,
                                                            T.replica, T.rs2);
        __syncthreads();
      }
    }
  }
}

// Spin half-steps of a small system: one workgroup holds every spin in LDS and
// runs the sweeps' classes one after another with barriers between them. A class
// of a few hundred atoms costs a launch of its own 3.3 us, most of it dispatch and
// two trips to memory; here the neighbours' spins are in LDS and the list entries
// and coefficients (from the exchange cache or the pair table) in L2. What bounds
// a piece of 512 atoms is one compute unit's LDS and L1 bandwidth (FP64: 1500
// clocks each). Two wavefronts per 64 atoms (four: 42 us instead of 28 per step of
// 2000 frozen atoms, FP32). Fetching ahead pays in FP32 (28 us instead of 30; with
// the bath and motion 72 instead of 85) and not in FP64 (41 instead of 36),
// where the two sets of coefficients leave too few of the 128 registers.
// Even half-steps use the positions of S, odd ones those of S2. With `same` the last
// update of a half-step and the first of the next, both of class 0, are one pass over it.
constexpr int kLdsLanes = 2, kLdsTeams = 16 / kLdsLanes;
template <typename real>
struct LdsSeq {
  const SpinLdsArgs &A;
  const float4 *tab2;  // at the positions of the odd half-steps
  const real *jc2;
  int hf, q, base;
  bool both;  // a class 0 pass over two half-steps
  __device__ int cls() const { return q < A.K ? q : 2 * A.K - 2 - q; }
  __device__ bool more() const { return hf < A.nhalf; }
  __device__ int begin() const { return base; }
  __device__ int end() const { return A.off[cls() + 1]; }
  __device__ int nrep() const { return q == A.K - 1 || both ? 2 : 1; }
  __device__ int64_t step(int r) const { return A.step + ((hf + (both ? r : 0)) >> 1); }
  __device__ int sub(int r) const {
    if (both) return r ? 2 * ((hf + 1) & 1) : 2 * (hf & 1) + 1;
    return 2 * (hf & 1) + (q < A.K ? r : 1);
  }
  __device__ const float4 *tab(const SysView<real> &S) const { return hf & 1 ? tab2 : S.tab; }
  __device__ const real *jc(const SysView<real> &S) const { return hf & 1 ? jc2 : S.jc; }
  __device__ void enter() {
    both = A.same && A.K > 1 && q == 2 * A.K - 2 && hf + 1 < A.nhalf;
    base = A.off[cls()];
  }
  __device__ void advance() {
    base += 64 * kLdsTeams;
    if (base < end()) return;
    if (++q > 2 * A.K - 2) {
      q = both ? 1 : 0;
      ++hf;
    }
    enter();
  }
  __device__ LdsSeq(const SpinLdsArgs &a, const SysView<real> &S2)
      : A(a), tab2(S2.tab), jc2(S2.jc), hf(0), q(0) {
    enter();
  }
  __device__ LdsSeq(const LdsSeq &o) = default;
  __device__ LdsSeq &operator=(const LdsSeq &o) {
    hf = o.hf;
    q = o.q;
    base = o.base;
    both = o.both;
    return *this;
  }
};
template <typename real, bool LANGEVIN, bool ANISO, int MLP>
__global__ __launch_bounds__(1024) void k_spin_lds(SysView<real> S, PotConst P, SpinLdsArgs A,
                                                   SysView<real> S2) {
  __shared__ real spin[3][sizeof(real) == 8 ? kLdsSpins64 : kLdsSpins32];
  __shared__ SpinTeam<real, kLdsLanes, 3, LANGEVIN ? 2 : 1> team[kLdsTeams];
  for (int i = threadIdx.x; i < S.n; i += 1024) {
    spin[0][i] = S.sx[i];
    spin[1][i] = S.sy[i];
    spin[2][i] = S.sz[i];
  }
  __syncthreads();
  if constexpr (sizeof(real) == 4) {
    spin_sequence<real, LANGEVIN, ANISO, kLdsLanes, kLdsTeams, MLP>(LdsSeq<real>(A, S2), S, P, spin[0], spin[1],
                                                                    spin[2], team, A.h, A.amp, A.seed,
                                                                    A.replica, A.rs2);
  } else {
    const int t = wave_id() / kLdsLanes, w = wave_id() % kLdsLanes;
    SysView<real> V = S;
    V.sx = spin[0];
    V.sy = spin[1];
    V.sz = spin[2];
    for (LdsSeq<real> q(A, S2); q.more(); q.advance()) {
      V.tab = q.tab(S);
      V.jc = q.jc(S);
      const int i = q.begin() + 64 * t + (int)(threadIdx.x & 63);
      const int64_t st[kMaxRep] = {q.step(0), q.step(1), 0, 0};
      const int sb[kMaxRep] = {q.sub(0), q.sub(1), 0, 0};
      spin_update<real, LANGEVIN, ANISO, kLdsLanes, MLP>(V, P, i, i < q.end(), w, team + t, q.nrep(), st, sb,
                                                         A.h, A.amp, A.seed, A.replica, A.rs2);
      __syncthreads();
    }
  }
  for (int i = threadIdx.x; i < S.n; i += 1024) {
    S.sx[i] = spin[0][i];
    S.sy[i] = spin[1][i];
    S.sz[i] = spin[2][i];
  }
}

// Exchange coefficients at one set of positions (the optional pair
// coefficient cache): J(r_ij) for every spin-segment entry, with the same
// expression as the spin phase's own evaluation. Positions change only at
// the drift, so one evaluation serves the two spin half-steps that use
// these positions (Sec. 3: coefficients must be re-evaluated after the
// positions move, and only then).
template <typename real, bool SPL>
__global__ __launch_bounds__(kBlock) void k_jcache(SysView<real> S, PotConst P, real *out,
                                                   double rs2, const int2 *tiles, int slots) {
  // with a tile table, block b takes the atom range of entry b (one spatial
  // slab of every class per XCD, as in the force launch)
  int i, end;
  if (tiles) {
    const int2 rg = tiles[blockIdx.x];
    i = rg.x + (int)threadIdx.x;
    end = rg.y;
  } else {
    i = blockIdx.x * blockDim.x + threadIdx.x;
    end = S.n;
  }
  if (i >= end) return;
  // grid.y splits the row into groups of `slots` slots: one group of all in a
  // large system; in a small one (few wavefronts per SIMD) a group is one
  // round, so that the row's rounds run side by side
  const int kb = (int)blockIdx.y * slots;
  const int ns = min(S.nspin[i], kb + slots);
  const double rix = S.rx[i], riy = S.ry[i], riz = S.rz[i];
  // slots in chunks of SL_JC_CHUNK with all loads of a chunk issued before
  // use (the row's own slots only: ns <= kcap)
  constexpr int CH = SL_JC_CHUNK;
  for (int k0 = kb; k0 < ns; k0 += CH) {
    int jj[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = k0 + c;
      const int j = k < ns ? S.nbr[(size_t)k * S.ld + i] : i;
      jj[c] = (unsigned)j < (unsigned)S.n ? j : i;
    }
    double xj[CH], yj[CH], zj[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      xj[c] = S.rx[jj[c]];
      yj[c] = S.ry[jj[c]];
      zj[c] = S.rz[jj[c]];
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int k = k0 + c;
      if (k >= ns) break;
      const double dx = min_image(rix - xj[c], S.L[0], S.invL[0]);
      const double dy = min_image(riy - yj[c], S.L[1], S.invL[1]);
      const double dz = min_image(riz - zj[c], S.L[2], S.invL[2]);
      const double r2 = dx * dx + dy * dy + dz * dz;
      if (SPL) {  // learned potential (spline form): J with its own cut
        out[(size_t)k * S.ld + i] = (real)spline_phys(S.spl, (float)sqrt(r2)).x;
      } else {
        out[(size_t)k * S.ld + i] = r2 < rs2 ? exch_J<real>(P, r2) : (real)0;
      }
    }
  }
}

template <typename real>
void launch_jcache(const SysView<real> &S, const PotConst &P, real *out, double rs2,
                   const int2 *tiles, int ntiles, int max_slots, hipStream_t st) {
  if (S.n <= 0) return;
  const int nx = tiles ? ntiles : (S.n + kBlock - 1) / kBlock;
  const bool split = S.n < kJcSplitAtoms && max_slots > SL_JC_CHUNK;
  const int slots = split ? slots_per_group(max_slots, SL_JC_CHUNK) : INT_MAX / 2;
  const dim3 grid(nx, split ? (max_slots + slots - 1) / slots : 1);
  if (S.spl.t) hipLaunchKernelGGL((k_jcache<real, true>), grid, dim3(kBlock), 0, st, S, P, out, rs2, tiles, slots);
  else hipLaunchKernelGGL((k_jcache<real, false>), grid, dim3(kBlock), 0, st, S, P, out, rs2, tiles, slots);
}
template void launch_jcache<double>(const SysView<double> &, const PotConst &, double *, double,
                                    const int2 *, int, int, hipStream_t);
template void launch_jcache<float>(const SysView<float> &, const PotConst &, float *, double,
                                   const int2 *, int, int, hipStream_t);

// Fixed-order sum of nb partial rows of 8 doubles (deterministic result).
__global__ __launch_bounds__(256) void k_reduce8(const double *partial, int nb, double *out) {
  __shared__ double buf[256][8];
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nb; b += 256)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] += partial[(size_t)b * 8 + c];
#pragma unroll
  for (int c = 0; c < 8; ++c) buf[threadIdx.x][c] = acc[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
#pragma unroll
      for (int c = 0; c < 8; ++c) buf[threadIdx.x][c] += buf[threadIdx.x + w][c];
    __syncthreads();
  }
  if (threadIdx.x < 8) out[threadIdx.x] = buf[0][threadIdx.x];
}


// ---------------------------------------------------------------------------
// Host launchers. The learned-potential variants (table lookups instead of
// the analytic J and V) exist in the FP32 form only; variant 4 is the
// analytic potential with the spin-orbit pair terms.
template <typename real, bool LG, bool AN, int LANES, int MLP, bool DUAL>
static void spin_phase_run(const SysView<real> &S, const PotConst &P, const SpinPhaseArgs &A,
                           const SysView<real> &S2, hipStream_t st) {
  using T = TeamShape<LANES, LG>;
  const int nb = (A.end - A.begin + T::atoms - 1) / T::atoms;
  const void *p[4] = {S.rx, S.ry, S.rz, S.sx};
  if (MLP == 1 || MLP == 3) {
    p[0] = MLP == 3 ? (const void *)S.jc : (const void *)S.tab;
    p[1] = S.sx;
    p[2] = S.sy;
    p[3] = S.sz;
  }
  SecondView<real, DUAL> V2;
  if constexpr (DUAL) V2 = S2;
  hipLaunchKernelGGL((k_spin_phase<real, LG, AN, LANES, MLP, DUAL>), dim3(nb), dim3(64 * T::waves), 0,
                     st, S.nbr, p[0], p[1], p[2], p[3], A.begin, A.end, S.ld, S.kcap, S, P, A, V2);
}

template <typename real, int LANES, int MLP, bool DUAL>
static void spin_phase_lanes3(const SysView<real> &S, const PotConst &P, const SpinPhaseArgs &A,
                              const SysView<real> &S2, hipStream_t st) {
  const bool lg = P.langevin != 0, an = P.aniso_on != 0;
  if (lg && an) spin_phase_run<real, true, true, LANES, MLP, DUAL>(S, P, A, S2, st);
  else if (lg) spin_phase_run<real, true, false, LANES, MLP, DUAL>(S, P, A, S2, st);
  else if (an) spin_phase_run<real, false, true, LANES, MLP, DUAL>(S, P, A, S2, st);
  else spin_phase_run<real, false, false, LANES, MLP, DUAL>(S, P, A, S2, st);
}

template <typename real, int LANES, int MLP>
static void spin_phase_lanes2(const SysView<real> &S, const PotConst &P, const SpinPhaseArgs &A,
                              const SysView<real> *S2, hipStream_t st) {
  if (S2) spin_phase_lanes3<real, LANES, MLP, true>(S, P, A, *S2, st);
  else spin_phase_lanes3<real, LANES, MLP, false>(S, P, A, S, st);
}

template <typename real, int LANES>
static void spin_phase_lanes(const SysView<real> &S, const PotConst &P, const SpinPhaseArgs &A,
                             const SysView<real> *S2, hipStream_t st) {
  constexpr bool f32 = sizeof(real) == 4;
  switch (spin_variant(S, P, S2)) {
    case 4: spin_phase_lanes2<real, LANES, 4>(S, P, A, S2, st); break;
    case 3: spin_phase_lanes2<real, LANES, 3>(S, P, A, S2, st); break;
    case 2: spin_phase_lanes2<real, LANES, (f32 ? 2 : 0)>(S, P, A, S2, st); break;
    case 1: spin_phase_lanes2<real, LANES, (f32 ? 1 : 0)>(S, P, A, S2, st); break;
    default: spin_phase_lanes2<real, LANES, 0>(S, P, A, S2, st); break;
  }
}

template <typename real>
void launch_spin_phase(const SysView<real> &S, const PotConst &P, const SpinPhaseArgs &A,
                       int lanes, hipStream_t st, const SysView<real> *S2) {
  if (A.end - A.begin <= 0) return;
  switch (lanes) {
    case 1: spin_phase_lanes<real, 1>(S, P, A, S2, st); break;
    case 2: spin_phase_lanes<real, 2>(S, P, A, S2, st); break;
    case 8: spin_phase_lanes<real, 8>(S, P, A, S2, st); break;
    default: spin_phase_lanes<real, 4>(S, P, A, S2, st); break;
  }
}

template <typename real, int LANES, int MLP>
static void spin_tail_run(const SysView<real> &S, const PotConst &P, const TailArgs &T,
                          hipStream_t st) {
  const bool lg = P.langevin != 0, an = P.aniso_on != 0;
  if (lg && an) hipLaunchKernelGGL((k_spin_tail<real, true, true, LANES, MLP>), dim3(1), dim3((kTailThreads<real, LANES, MLP>)), 0, st, S, P, T);
  else if (lg) hipLaunchKernelGGL((k_spin_tail<real, true, false, LANES, MLP>), dim3(1), dim3((kTailThreads<real, LANES, MLP>)), 0, st, S, P, T);
  else if (an) hipLaunchKernelGGL((k_spin_tail<real, false, true, LANES, MLP>), dim3(1), dim3((kTailThreads<real, LANES, MLP>)), 0, st, S, P, T);
  else hipLaunchKernelGGL((k_spin_tail<real, false, false, LANES, MLP>), dim3(1), dim3((kTailThreads<real, LANES, MLP>)), 0, st, S, P, T);
}

template <typename real, int MLP>
static void spin_tail_lanes(const SysView<real> &S, const PotConst &P, const TailArgs &T, hipStream_t st) {
  int m = 0, reps = 0;
  for (int q = 0; q < T.nitems; ++q) {
    m = std::max(m, T.item[q].end - T.item[q].begin);
    reps = std::max(reps, T.item[q].nrep);
  }
  if constexpr (MLP != 4)
    if (m > kTailBlock / kTailLanes && reps <= kTailWide) return spin_tail_run<real, kTailWide, MLP>(S, P, T, st);
  spin_tail_run<real, kTailLanes, MLP>(S, P, T, st);
}

template <typename real>
void launch_spin_tail(const SysView<real> &S, const PotConst &P, const TailArgs &T, hipStream_t st) {
  if (T.nitems <= 0) return;
  constexpr bool f32 = sizeof(real) == 4;
  switch (spin_variant<real>(S, P, nullptr)) {
    case 4: spin_tail_lanes<real, 4>(S, P, T, st); break;
    case 3: spin_tail_lanes<real, 3>(S, P, T, st); break;
    case 2: spin_tail_lanes<real, (f32 ? 2 : 0)>(S, P, T, st); break;
    case 1: spin_tail_lanes<real, (f32 ? 1 : 0)>(S, P, T, st); break;
    default: spin_tail_lanes<real, 0>(S, P, T, st); break;
  }
}

template <typename real, int MLP>
static void spin_lds_run(const SysView<real> &S, const PotConst &P, const SpinLdsArgs &A,
                         const SysView<real> &S2, hipStream_t st) {
  const bool lg = P.langevin != 0, an = P.aniso_on != 0;
  if (lg && an) hipLaunchKernelGGL((k_spin_lds<real, true, true, MLP>), dim3(1), dim3(1024), 0, st, S, P, A, S2);
  else if (lg) hipLaunchKernelGGL((k_spin_lds<real, true, false, MLP>), dim3(1), dim3(1024), 0, st, S, P, A, S2);
  else if (an) hipLaunchKernelGGL((k_spin_lds<real, false, true, MLP>), dim3(1), dim3(1024), 0, st, S, P, A, S2);
  else hipLaunchKernelGGL((k_spin_lds<real, false, false, MLP>), dim3(1), dim3(1024), 0, st, S, P, A, S2);
}

template <typename real>
bool launch_spin_lds(const SysView<real> &S, const PotConst &P, const SpinLdsArgs &A,
                     const SysView<real> &S2, hipStream_t st) {
  if (S.n > (sizeof(real) == 8 ? kLdsSpins64 : kLdsSpins32) || P.soc_on) return false;
  if (S.jc && S2.jc) spin_lds_run<real, 3>(S, P, A, S2, st);
  else if (sizeof(real) == 4 && S.tab && S2.tab) spin_lds_run<real, (sizeof(real) == 4 ? 1 : 3)>(S, P, A, S2, st);
  else return false;
  return true;
}
template bool launch_spin_lds<double>(const SysView<double> &, const PotConst &, const SpinLdsArgs &,
                                      const SysView<double> &, hipStream_t);
template bool launch_spin_lds<float>(const SysView<float> &, const PotConst &, const SpinLdsArgs &,
                                     const SysView<float> &, hipStream_t);

void launch_reduce8(const double *partial, int nb, double *out, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce8, dim3(1), dim3(256), 0, st, partial, nb, out);
}


template void launch_spin_phase<double>(const SysView<double> &, const PotConst &,
                                        const SpinPhaseArgs &, int, hipStream_t,
                                        const SysView<double> *);
template void launch_spin_phase<float>(const SysView<float> &, const PotConst &,
                                       const SpinPhaseArgs &, int, hipStream_t,
                                       const SysView<float> *);
template void launch_spin_tail<double>(const SysView<double> &, const PotConst &,
                                       const TailArgs &, hipStream_t);
template void launch_spin_tail<float>(const SysView<float> &, const PotConst &, const TailArgs &,
                                      hipStream_t);

}  // namespace sl
