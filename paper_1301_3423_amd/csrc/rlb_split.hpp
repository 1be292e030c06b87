// The time step with the populations of a cell split over the wavefronts of
// a workgroup, for work too small to fill the chip with whole cells.  There
// a step lasts as long as one wavefront's chain of instructions (a lane that
// holds a whole cell, or half of one, issues over 4000: 8-10 us at one
// wavefront per SIMD, whatever the number of cells), so the chain is cut:
//
// A workgroup of NG wavefronts works on 64 consecutive cells, one per lane.
// Wavefront g holds a run of inversion pairs of one energy shell (Groups) of
// all 64 cells: it gathers them, forms their ShellSums, and once the frame is
// known relaxes and stores them.  The sums meet in LDS (10 doubles per lane
// and wavefront, one barrier) and every wavefront adds them up in the same
// order; the Landau solve and tau are computed by every wavefront for itself.
#pragma once

#include "rlb_kernels.hpp"

namespace rlb {

// The inversion pairs [begin(g), begin(g + 1)) of group g.  float32: one
// group per shell, so that the shells' sums are those of the one-lane
// kernels, bit for bit.  float64: four (third order) or three groups of
// nearly equal size, whichever shells they meet, which share their part of
// the 14 moments.
template <class M, class S>
struct Split {
  static constexpr bool by_shell = sizeof(S) == 4;
  static constexpr int NG = M::NSHELL;
  static constexpr int begin(int g) { return by_shell ? shell_pair_begin<M>(g) : M::Q / 2 * g / NG; }
  static constexpr int max_pairs() {
    int m = 0;
    for (int g = 0; g < NG; ++g) m = begin(g + 1) - begin(g) > m ? begin(g + 1) - begin(g) : m;
    return m;
  }
  static constexpr int N = 2 * max_pairs();
  using Pops = S[N]; // the populations a lane holds
  static constexpr int SHARE = by_shell ? 10 : 14;
  // the pairs of group g in shell l
  static constexpr int seg_begin(int g, int l) {
    return shell_pair_begin<M>(l) > begin(g) ? shell_pair_begin<M>(l) : begin(g);
  }
  static constexpr int seg_end(int g, int l) {
    return shell_pair_begin<M>(l + 1) < begin(g + 1) ? shell_pair_begin<M>(l + 1) : begin(g + 1);
  }
};
static_assert(sizeof(ShellSums) == 10 * sizeof(double) && sizeof(Moments) == 14 * sizeof(double));

// What group G adds to the moments, from its members f (2k at 2 (k - begin),
// 2k + 1 after it), left for the other wavefronts in part[G].
template <class M, class S, int G>
__device__ __forceinline__ void share_sums(const typename Split<M, S>::Pops &f, double (*part)[Split<M, S>::SHARE][64],
                                           int lane) {
  using D = Split<M, S>;
  constexpr int K0 = D::begin(G);
  Moments m{};
  const double *src = &m.N0;
  ShellSums a;
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value, kb = D::seg_begin(G, l), ke = D::seg_end(G, l);
    if constexpr (kb < ke) {
      a = ShellSums{};
      static_for<kb, ke>([&](auto K) {
        constexpr int k = decltype(K)::value;
        const double x = static_cast<double>(f[2 * (k - K0)]);
        const double y = static_cast<double>(f[2 * (k - K0) + 1]);
        a.template add_pair<M, k>(x + y, x - y);
        a.pin();
      });
      if constexpr (D::by_shell)
        src = &a.sh;
      else
        a.template fold<M, l>(m);
    }
  });
#pragma unroll
  for (int j = 0; j < D::SHARE; ++j) part[G][j][lane] = src[j];
}

// The moments of the lane's cell from the shares of all groups, in their
// order (after a barrier).
template <class M, class S>
__device__ __forceinline__ Moments gathered_moments(const double (*part)[Split<M, S>::SHARE][64], int lane) {
  using D = Split<M, S>;
  Moments m{};
  if constexpr (D::by_shell) {
    static_for<0, M::NSHELL>([&](auto L) {
      constexpr int l = decltype(L)::value;
      ShellSums t;
      double *dst = &t.sh;
#pragma unroll
      for (int j = 0; j < D::SHARE; ++j) dst[j] = part[l][j][lane];
      t.template fold<M, l>(m);
    });
  } else {
    double *dst = &m.N0;
#pragma unroll
    for (int j = 0; j < D::SHARE; ++j) {
      dst[j] = part[0][j][lane];
#pragma unroll
      for (int g = 1; g < D::NG; ++g) dst[j] += part[g][j][lane];
    }
  }
  return m;
}

// Equilibrium and relaxation of the pairs of group G (relax_cell's
// arithmetic); post-collision values replace f.
template <class M, class S, int G>
__device__ __forceinline__ void relax_group(typename Split<M, S>::Pops &f, const EqCoef<M> &e, const Frame &fr, double tau) {
  using CT = S;
  using D = Split<M, S>;
  constexpr int K0 = D::begin(G);
  const double g = fr.U0 / tau;
  const CT gg = CT(g);
  const CT bx = CT(g * fr.vx * M::INV_R), by = CT(g * fr.vy * M::INV_R), bz = CT(g * fr.vz * M::INV_R);
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value, kb = D::seg_begin(G, l), ke = D::seg_end(G, l);
    if constexpr (kb < ke) {
      const ShellCoef<M, CT> s = shell_coefficients<M, l, CT>(e);
      static_for<kb, ke>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr Point P = M::P[2 * k];
        CT E, O;
        shell_eval<M, 2 * k, CT>(s, E, O);
        const CT wE = CT(P.w) * E, wO = CT(P.w) * O;
        CT t = CT(0);
        if constexpr (P.tx != 0) t = fmadd(CT(P.tx), bx, t);
        if constexpr (P.ty != 0) t = fmadd(CT(P.ty), by, t);
        if constexpr (P.tz != 0) t = fmadd(CT(P.tz), bz, t);
        S &a = f[2 * (k - K0)], &b = f[2 * (k - K0) + 1];
        a = fmadd(gg - t, (wE + wO) - a, a);
        b = fmadd(gg + t, (wE - wO) - b, b);
      });
      __builtin_amdgcn_sched_barrier(0); // one shell's coefficients live at a time
    }
  });
}

// Calls f(integral_constant<int, G>) for the wavefront's own group.
template <int NG, int G = 0, class F>
__device__ __forceinline__ void for_group(int grp, F &&f) {
  if constexpr (G + 1 < NG) {
    if (grp == G)
      f(std::integral_constant<int, G>{});
    else
      for_group<NG, G + 1>(grp, f);
  } else {
    f(std::integral_constant<int, G>{});
  }
}

// ---- several steps of many tubes in one launch -------------------------------
//
// Each launch takes every tube `ksteps` steps further (or what it has left).
// A workgroup works on 64 consecutive cells of one tube: after k steps the
// 64 - 12 (k - 1) cells in the middle are right (a step reaches at most MAXD
// cells), and only those are stored; between steps the populations move from
// lane to lane, along z, without leaving the registers.  So a launch reads
// and writes memory once for its k steps, and the cost of starting it
// (3.8 us from one empty kernel to the next) and of the loads is shared by
// them; more steps mean more cells computed twice, so the host picks k.
// A 1600-cell float64 tube takes 5.6 us per step with k = 5 (8.2 with k = 1;
// 74 as one workgroup of k_tubes, one of 256 CUs), 24 tubes of 200-4000 cells
// 28 us with k = 2 (196), 96 of them 109 (224); mixed 5.1 (37), 18 (96) and
// 59 us (112).  What bounds it: the chain of one wavefront (776 float64
// instructions of the moments' sum, the frame and the coefficients, 610 of
// its group), 4.4 us per step; with more tiles than CUs, the arithmetic.
inline constexpr int TUBE_TILE = 64;
constexpr int tube_tile_cells(int k) { return TUBE_TILE - 2 * MAXD * (k - 1); }
inline constexpr int TUBE_MAX_KSTEPS = 5;
static_assert(tube_tile_cells(TUBE_MAX_KSTEPS) > 0);

// The value `v` of lane (l - shift) mod 64.
__device__ __forceinline__ float from_lane(float v, int addr) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double from_lane(double v, int addr) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(addr, static_cast<int>(u & 0xffffffffu)));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(addr, static_cast<int>(u >> 32)));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Third-order float64 takes one wavefront per SIMD, whose 328 registers hold
// everything (with two per SIMD the compiler spills 200 registers: 7.9
// instead of 5.6 us per step of a 1600-cell tube, 35 instead of 28 of 24).
template <class M, class S>
inline constexpr int tile_waves = sizeof(S) == 8 && M::Q == 128 ? 1 : 2;

// desc[0 .. ntubes): the tubes of this launch, steps = steps left before
// round 0, spin_limit = index of the tube's first tile; id[k]: where tube k's
// status lies.  Round `round` of the launches reads buffer (cur + round) & 1.
template <class M, class S>
__global__ void __launch_bounds__(64 * (Split<M, S>::NG)) __attribute__((amdgpu_waves_per_eu(tile_waves<M, S>)))
k_tubes_tile(S *__restrict__ base, const TubeDesc *__restrict__ desc, const int *__restrict__ id, int ntubes,
             int round, int ksteps, unsigned *__restrict__ status) {
  using D = Split<M, S>;
  constexpr int NG = D::NG;
  constexpr int T = TILE<S>;
  __shared__ double part[2][NG][D::SHARE][64];
  const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int tile = static_cast<int>(blockIdx.x);
  // the last tube whose first tile is <= tile: 64 candidates at a time
  int j = 0;
  for (int span = ntubes; span > 1;) {
    const int stride = (span + 63) / 64;
    const int q = j + lane * stride;
    const bool below = lane * stride < span && desc[q < ntubes ? q : ntubes - 1].spin_limit <= tile;
    const int hits = __popcll(__ballot(below));
    j += (hits - 1) * stride;
    const int left = span - (hits - 1) * stride;
    span = left < stride ? left : stride;
  }
  j = __builtin_amdgcn_readfirstlane(j);
  const TubeDesc d = desc[j];
  const int64_t left = d.steps - static_cast<int64_t>(round) * ksteps;
  const int k = left < ksteps ? static_cast<int>(left) : ksteps;
  if (k <= 0) return;
  const int cells = tube_tile_cells(ksteps);
  const int h = MAXD * (k - 1);
  const int c0 = (tile - d.spin_limit) * cells;
  const int n = d.n;
  int z = (c0 - h + lane) % n;
  if (z < 0) z += n;
  const bool store = lane >= h && lane < h + cells && c0 + lane - h < n;
  const int cur = (d.cur + round) & 1;
  const S *in = base + (cur ? d.off[1] : d.off[0]);
  S *out = base + (cur ? d.off[0] : d.off[1]);
  Relax rx;
  rx.mode = d.mode;
  rx.tau = d.tau;
  rx.eta_s = d.eta_s;
  int zo[2 * MAXD + 1];
#pragma unroll
  for (int s = -MAXD; s <= MAXD; ++s) zo[s + MAXD] = static_cast<int>(tile_elem<M, S>(wrap_back(z, s, n)));
  typename D::Pops f;
  for_group<NG>(grp, [&](auto G) {
    constexpr int q = decltype(G)::value;
    constexpr int I0 = 2 * D::begin(q), I1 = 2 * D::begin(q + 1);
    static_for<I0, I1>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr Point P = M::P[i];
      f[i - I0] = load_at(in + i * T, zo[P.tz + MAXD]);
    });
    __builtin_amdgcn_sched_barrier(0);
    share_sums<M, S, q>(f, part[0], lane);
  });
  unsigned flags = 0;
  for (int s = 0;; ++s) {
    // the barrier also keeps the writers of part[s & 1], two steps later, behind its readers
    __syncthreads();
    const Moments m = gathered_moments<M, S>(part[s & 1], lane);
    Frame fr{1.0, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (lane >= MAXD * s && lane < TUBE_TILE - MAXD * s) flags |= landau_frame(m, fr);
    const double tau = relaxation_time<M>(rx, fr.n, fr.T);
    const EqCoef<M> e = eq_coefficients<M>(fr.n, fr.T, fr.U0, fr.Ux, fr.Uy, fr.Uz);
    const bool last = s + 1 == k;
    for_group<NG>(grp, [&](auto G) {
      constexpr int q = decltype(G)::value;
      constexpr int I0 = 2 * D::begin(q), I1 = 2 * D::begin(q + 1);
      relax_group<M, S, q>(f, e, fr, tau);
      if (last) {
        // fresh copies keep the compiler from forming every address before the loop
        int o = static_cast<int>(tile_elem<M, S>(z));
        int zero = 0;
        asm volatile("" : "+v"(o), "+s"(zero));
        S *dst = out + zero;
        if (store)
          static_for<I0, I1>([&](auto I) {
            constexpr int i = decltype(I)::value;
            store_plain(dst + i * T, o, f[i - I0]);
          });
      } else {
        int l = lane;
        asm volatile("" : "+v"(l));
        static_for<I0, I1>([&](auto I) {
          constexpr int i = decltype(I)::value;
          if constexpr (M::P[i].tz != 0) f[i - I0] = from_lane(f[i - I0], (l - M::P[i].tz) * 4);
        });
        share_sums<M, S, q>(f, part[(s + 1) & 1], lane);
      }
    });
    if (last) break;
  }
  if (flags && grp == 0) atomicOr(status + id[j], flags);
}

} // namespace rlb
