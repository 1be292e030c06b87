// The time step with the populations of a cell split over two wavefronts, for
// tubes and small boxes.  A lane that holds a whole cell (or half of one)
// issues over 4000 instructions per step: 8-10 us at one wavefront per SIMD,
// however few cells there are.  Here the chain is cut:
//
// A workgroup of two wavefronts works on 64 consecutive cells (float32, one
// cell per lane) or 32 (float64, one on lanes c and c + 32, as in k_step).
// Each wavefront holds the points of its own shells (Split): it gathers them,
// sums them up per shell and, once the frame is known, relaxes and stores them.
// The sums meet in wavefront 0, which solves for the frame while the other
// waits (and leaves the SIMD to other workgroups); tau and the coefficients of
// the equilibrium are dealt out again, by parity block, and meet in LDS.  Three
// barriers per step.  Every sum is formed in the order of the unsplit kernels
// (k_step in float64, k_tubes in both), so the bits are theirs.
//
// Why two wavefronts and 32 KB of LDS and not more: a workgroup is placed only
// where all of it fits at once.  Beside kernels of 128-thread workgroups that
// keep the chip full (a large box on another stream) a workgroup of four
// wavefronts finds no place until they drain, one of two takes the place of any
// workgroup that ends.  200 float64 steps of a 32^3 box beside a 256^3 one: two-lane
// kernel 10.5 ms, split over four wavefronts 594, over two 11.5; 300 steps of 24 tubes
// of 200-4000 cells 637 and 18 ms, and with 36 KB of LDS, beside a float64 box, 114.
#pragma once

#include "rlb_kernels.hpp"

namespace rlb {

// Which shells a wavefront holds: group 0 or 1 of two nearly equal parts (third
// order 29 and 35 pairs, second order 18 and 15), or everything (NG = 1).
template <class M, class S, int NG>
struct Split {
  static_assert(NG == 1 || NG == 2);
  // float64: a cell on two lanes, each with one member of every pair
  static constexpr bool halves = sizeof(S) == 8;
  static constexpr int CELLS = halves ? 32 : 64; // of a workgroup
  static constexpr int MEMBERS = halves ? 1 : 2; // of a pair, on one lane
  static constexpr int owner(int l) { // the group of a shell
    constexpr int o3[4] = {0, 1, 1, 0}, o2[3] = {0, 0, 1};
    return NG == 1 ? 0 : M::ORDER == 3 ? o3[l] : o2[l];
  }
  static constexpr int size(int l) { return shell_pair_begin<M>(l + 1) - shell_pair_begin<M>(l); }
  // place of shell l among its group's
  static constexpr int nth(int l) {
    int n = 0;
    for (int i = 0; i < l; ++i) n += owner(i) == owner(l);
    return n;
  }
  // place of pair k of shell l among its group's pairs
  static constexpr int local(int l, int k) {
    int n = k - shell_pair_begin<M>(l);
    for (int i = 0; i < l; ++i)
      if (owner(i) == owner(l)) n += size(i);
    return n;
  }
  static constexpr int max_size() {
    int n[2] = {0, 0};
    for (int l = 0; l < M::NSHELL; ++l) n[owner(l)] += size(l);
    return n[0] > n[1] ? n[0] : n[1];
  }
  static constexpr int N = MEMBERS * max_size();
  using Pops = S[N]; // the populations a lane holds: pair k from MEMBERS * local(k)

  // f(shell, pair, its place) for the pairs of group G
  template <int G, class F>
  static __device__ __forceinline__ void pairs(F &&f) {
    static_for<0, M::NSHELL>([&](auto L) {
      constexpr int l = decltype(L)::value;
      if constexpr (owner(l) == G)
        static_for<shell_pair_begin<M>(l), shell_pair_begin<M>(l + 1)>([&](auto K) {
          f(L, K, std::integral_constant<int, MEMBERS * local(l, decltype(K)::value)>{});
        });
    });
  }
  // f(point, its place) for the points a lane of group G holds; with halves the
  // point is the pair's first, and the lane's own is the first or the second
  template <int G, class F>
  static __device__ __forceinline__ void points(F &&f) {
    pairs<G>([&](auto, auto K, auto P) {
      constexpr int i = 2 * decltype(K)::value, p = decltype(P)::value;
      f(std::integral_constant<int, i>{}, P);
      if constexpr (!halves) f(std::integral_constant<int, i + 1>{}, std::integral_constant<int, p + 1>{});
    });
  }
};

// What a workgroup's wavefronts hand each other, per lane or cell: 29 KB in
// float64 and 31 in float32 (third order), so that a workgroup also fits where one
// of the float64 step's (32 KB, k_step) ended.
template <class M, class S, int NG>
struct Shared {
  static constexpr int CELLS = Split<M, S, NG>::CELLS;
  static constexpr int SUMS = 10; // of a shell
  static constexpr int shells1() {
    int n = 0;
    for (int l = 0; l < M::NSHELL; ++l) n += Split<M, S, NG>::owner(l) == 1;
    return n;
  }
  double sums[shells1()][SUMS][64]; // of group 1's shells
  double frame[9][CELLS];           // n, T, U0, Ux, Uy, Uz, vx, vy, vz
  double rate[CELLS];               // gamma / tau
  S coef[M::NSHELL][SpatialTable<M>::NS][CELLS];
};
template <class M, class S>
struct Shared<M, S, 1> {}; // a wavefront that holds whole cells
static_assert(sizeof(Shared<M3, double, 2>) <= 32768 && sizeof(Shared<M3, float, 2>) <= 32768);
static_assert(sizeof(ShellSums) == 10 * sizeof(double));

// The sums of group G's shells: group 0 keeps them (own[shell]), group 1
// leaves them in LDS.
template <class D, class M, int G, class W>
__device__ __forceinline__ void shell_sums(const typename D::Pops &f, ShellSums (&own)[M::NSHELL], W &w, int lane) {
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value;
    if constexpr (D::owner(l) == G) {
      ShellSums a{};
      static_for<shell_pair_begin<M>(l), shell_pair_begin<M>(l + 1)>([&](auto K) {
        constexpr int k = decltype(K)::value, p = D::MEMBERS * D::local(l, k);
        const double x = static_cast<double>(f[p]);
        if constexpr (D::halves) {
          a.template add_pair<M, k>(x, x);
        } else {
          const double y = static_cast<double>(f[p + 1]);
          a.template add_pair<M, k>(x + y, x - y);
        }
        a.pin();
      });
      if constexpr (G == 0) {
        own[l] = a;
      } else {
        const double *src = &a.sh;
#pragma unroll
        for (int j = 0; j < W::SUMS; ++j) w.sums[D::nth(l)][j][lane] = src[j];
      }
    }
  });
}

// Group 0, after a barrier: the moments of the lane's cell from the sums of
// all shells, in their order.
template <class D, class M, class W>
__device__ __forceinline__ Moments gathered_moments(const ShellSums (&own)[M::NSHELL], const W &w, int lane) {
  Moments m{};
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value;
    if constexpr (D::owner(l) == 0) {
      own[l].template fold<M, l>(m);
    } else {
      ShellSums t;
      double *dst = &t.sh;
#pragma unroll
      for (int j = 0; j < W::SUMS; ++j) dst[j] = w.sums[D::nth(l)][j][lane];
      t.template fold<M, l>(m);
    }
  });
  if constexpr (D::halves) return both_members(m, lane < 32 ? 1.0 : -1.0);
  return m;
}

template <class W>
__device__ __forceinline__ void share_frame(const Frame &fr, W &w, int cell) {
  const double v[9] = {fr.n, fr.T, fr.U0, fr.Ux, fr.Uy, fr.Uz, fr.vx, fr.vy, fr.vz};
#pragma unroll
  for (int j = 0; j < 9; ++j) w.frame[j][cell] = v[j];
}

// The wavefront that computes a parity block of the equilibrium's coefficients
// (blocks of 8, 5, 5, 5, 2, 2, 2 and 1, or 5, 2, 2, 2, 1, 1, 1); wavefront 0
// has tau to compute as well.
template <class M>
constexpr int block_owner(int b) {
  constexpr int o3[8] = {1, 0, 1, 1, 0, 0, 0, 0}, o2[7] = {1, 1, 1, 0, 0, 0, 0};
  return M::ORDER == 3 ? o3[b] : o2[b];
}

// After a barrier behind share_frame.  Group 0: the relaxation rate; group G:
// the coefficients of its blocks in the theta-polynomials of every shell
// (eq_coefficients and shell_coefficients, operation for operation).
template <class D, class M, class S, int G, class W>
__device__ __forceinline__ void share_coefficients(const Relax &rx, W &w, int cell) {
  const double n = w.frame[0][cell], T = w.frame[1][cell], U0 = w.frame[2][cell];
  const MJ mj = mj_of(n, T, U0, w.frame[3][cell], w.frame[4][cell], w.frame[5][cell]);
  if constexpr (G == 0) w.rate[cell] = U0 / relaxation_time<M>(rx, n, T);
  static_for<0, M::NBLOCK>([&](auto B) {
    constexpr int blk = decltype(B)::value;
    if constexpr (block_owner<M>(blk) == G) {
      constexpr int b0 = M::BLOCK_BEGIN[blk], b1 = M::BLOCK_BEGIN[blk + 1];
      const EqBlock<M, blk> e = eq_block<M, blk>(mj);
      static_for<0, SpatialTable<M>::NS>([&](auto Sx) {
        constexpr int si = decltype(Sx)::value;
        if constexpr (spatial_block<M>(si) == blk) {
          static_for<0, M::NSHELL>([&](auto L) {
            constexpr int l = decltype(L)::value;
            // (float64: both lanes of a cell write the same value)
            w.coef[l][si][cell] = S(spatial_coefficient<M, l, si, b0, b1>(e.c));
          });
        }
      });
    }
  });
}

// Equilibrium and relaxation of the points of group G (the arithmetic of
// relax_cell, or of the two-lane kernel); post-collision values replace f.
template <class D, class M, class S, int G, class W>
__device__ __forceinline__ void relax_group(typename D::Pops &f, const W &w, int lane) {
  using CT = S;
  const int cell = lane % D::CELLS;
  const double sg = D::halves && lane >= 32 ? -1.0 : 1.0;
  const double g = w.rate[cell];
  const CT gg = CT(g), sgn = CT(sg);
  const double gs = D::halves ? g * M::INV_R * sg : g;
  CT bx, by, bz;
  if constexpr (D::halves) {
    bx = CT(gs * w.frame[6][cell]), by = CT(gs * w.frame[7][cell]), bz = CT(gs * w.frame[8][cell]);
  } else {
    bx = CT(gs * w.frame[6][cell] * M::INV_R), by = CT(gs * w.frame[7][cell] * M::INV_R);
    bz = CT(gs * w.frame[8][cell] * M::INV_R);
  }
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value;
    if constexpr (D::owner(l) == G) {
      ShellCoef<M, CT> s;
#pragma unroll
      for (int si = 0; si < SpatialTable<M>::NS; ++si) s.c[si] = w.coef[l][si][cell];
      static_for<shell_pair_begin<M>(l), shell_pair_begin<M>(l + 1)>([&](auto K) {
        constexpr int k = decltype(K)::value, p = D::MEMBERS * D::local(l, k);
        constexpr Point P = M::P[2 * k];
        CT E, O;
        shell_eval<M, 2 * k, CT>(s, E, O);
        CT t = CT(0);
        if constexpr (P.tx != 0) t = fmadd(CT(P.tx), bx, t);
        if constexpr (P.ty != 0) t = fmadd(CT(P.ty), by, t);
        if constexpr (P.tz != 0) t = fmadd(CT(P.tz), bz, t);
        S &a = f[p];
        if constexpr (D::halves) {
          // E + sigma O is rounded once, as the sum of coefficients with their signs
          const CT feq = CT(P.w) * fmadd(sgn, O, E);
          a = fmadd(gg - t, feq - a, a);
        } else {
          S &b = f[p + 1];
          const CT wE = CT(P.w) * E, wO = CT(P.w) * O;
          a = fmadd(gg - t, (wE + wO) - a, a);
          b = fmadd(gg + t, (wE - wO) - b, b);
        }
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

// ---- one float64 step of a small box ------------------------------------------
//
// While the chip is not full a step lasts as long as a workgroup: the launch
// (3.8 us), the gathers' latency and one wavefront's chain, half of the two-lane
// kernel's (k_step), which a larger box keeps hidden behind its memory traffic.
// 1 x 1 x 1600 10.7 -> 8.2 us per step, 16^3 11.6 -> 9.0, 32^3 18.6 -> 15.6 (4.3 TB/s,
// from the caches).  Offsets are 32-bit; the 24-bit multiply that forms them
// matters (a 32-bit one cost 2 us at 32^3).
template <class M, bool WALLS, int AC>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2)))
k_step_split(InPtr<double, AC> cur, OutPtr<double, AC> nxt, Geom g, Relax rx, unsigned *__restrict__ status,
             const uint8_t *__restrict__ solid) {
  using S = double;
  using D = Split<M, S, 2>;
  constexpr int T = TILE<S>;
  __shared__ Shared<M, S, 2> w;
  const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int m = lane >> 5, sigma = 1 - 2 * m;
  int cell = pair_block_order(blockIdx.x, gridDim.x) * D::CELLS + (lane & 31);
  bool active = cell < g.cells;
  if (!active) cell = g.cells - 1; // computed, never stored
  if constexpr (WALLS) active = active && solid[cell] == 0;
  int x, y, z;
  cell_coords(cell, g, x, y, z);
  const HalfShifts sh(x, y, z, sigma, g);
  constexpr uint32_t SEG = T * sizeof(S); // bytes from a population to the next
  const uint32_t own = tile_bytes32<M, S>(cell);
  const uint32_t ms = static_cast<uint32_t>(m) * SEG, other = SEG - ms; // the slots of the own and of the inverse point
  const char *in = reinterpret_cast<const char *>(cur);
  char *out = reinterpret_cast<char *>(nxt);
  // a wavefront runs its own group's code from here to the end; each passes the
  // same barriers
  for_group<2>(grp, [&](auto G) {
    constexpr int q = decltype(G)::value;
    typename D::Pops f;
    D::template points<q>([&](auto I, auto P) {
      constexpr int i = decltype(I)::value;
      constexpr Point PT = M::P[i];
      const uint32_t o = AC == AA_EVEN ? own : tile_bytes32<M, S>(sh.template back<PT.tx, PT.ty, PT.tz>());
      f[decltype(P)::value] = *reinterpret_cast<const S *>(in + i * SEG + (o + (AC == AA_ODD ? other : ms)));
    });
    __builtin_amdgcn_sched_barrier(0);
    ShellSums mine[M::NSHELL]; // group 0
    shell_sums<D, M, q>(f, mine, w, lane);
    __syncthreads();
    unsigned flags = 0;
    if constexpr (q == 0) {
      Frame fr;
      flags = landau_frame(gathered_moments<D, M>(mine, w, lane), fr);
      share_frame(fr, w, lane & 31);
    }
    __syncthreads();
    share_coefficients<D, M, S, q>(rx, w, lane & 31);
    __syncthreads();
    relax_group<D, M, S, q>(f, w, lane);
    // in place, odd: to x + sigma theta; the offsets are formed here rather than
    // kept through the arithmetic
    int xs = x;
    asm volatile("" : "+v"(xs));
    const HalfShifts to(xs, y, z, -sigma, g);
    if (active) {
      D::template points<q>([&](auto I, auto P) {
        constexpr int i = decltype(I)::value, p = decltype(P)::value;
        constexpr Point PT = M::P[i];
        if constexpr (AC == AA_ODD)
          *reinterpret_cast<S *>(out + i * SEG + (tile_bytes32<M, S>(to.template back<PT.tx, PT.ty, PT.tz>()) + ms)) =
              f[p];
        else
          __builtin_nontemporal_store(
              f[p], reinterpret_cast<S *>(out + i * SEG + (own + (AC == AA_EVEN ? other : ms))));
      });
      if (flags) atomicOr(status, flags);
    }
  });
}

// ---- several steps of many tubes in one launch -------------------------------
//
// Each launch takes every tube `ksteps` steps further (or what it has left).
// A workgroup works on the 64 (float64: 32) consecutive cells of a tile of one
// tube: after k steps the middle ones, all but 6 (k - 1) on either side, are
// right (a step reaches at most MAXD cells), and only those are stored; between
// steps the populations move from lane to lane, along z, without leaving the
// registers.  So a launch reads and writes memory once for its k steps, and the
// cost of starting it (3.8 us from one empty kernel to the next) and of the
// loads is shared by them; more steps mean more cells computed twice, so the
// host picks k.
template <class S>
inline constexpr int TUBE_TILE = sizeof(S) == 8 ? 32 : 64;
template <class S>
constexpr int tube_tile_cells(int k) {
  return TUBE_TILE<S> - 2 * MAXD * (k - 1);
}
template <class S>
inline constexpr int TUBE_MAX_KSTEPS = sizeof(S) == 8 ? 3 : 5;
static_assert(tube_tile_cells<float>(TUBE_MAX_KSTEPS<float>) > 0 && tube_tile_cells<double>(TUBE_MAX_KSTEPS<double>) > 0);

// The value `v` of lane addr / 4 mod 64.
__device__ __forceinline__ float from_lane(float v, int addr) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double from_lane(double v, int addr) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(addr, static_cast<int>(u & 0xffffffffu)));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(addr, static_cast<int>(u >> 32)));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// The last of `ntubes` tubes whose first tile is <= tile.  Scalar loads of a
// few cache lines that all workgroups share: under load a vector load takes
// microseconds, and this comes before anything else can start.
__device__ __forceinline__ int tube_of_tile(const int *__restrict__ first, int ntubes, int tile) {
  int lo = 0;
  for (int hi = ntubes; hi - lo > 1;) {
    const int mid = (lo + hi) >> 1;
    if (first[mid] <= tile)
      lo = mid;
    else
      hi = mid;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// What bounds it.  Few tiles: the chain of one wavefront, 4.9 us per step (third
// order): the sums over its points, three barriers, the frame, tau or
// coefficients, its points' equilibrium.  A 200-cell float64 tube takes 5.8 us per
// step with k = 3 (7.8 with k = 1; as one workgroup per tube, k_tubes, 14.6), one of 1600
// cells 6.1 (74); mixed, k = 5, 5.6 (9.4) and 5.8 (37).  With more tiles than CUs, the
// arithmetic: 24 float64 tubes of 200-4000 cells 27 us with k = 2 (196), 512 of
// them 424 with k = 1 (433, little gain: 2.6e9 updates/s); mixed 12.5 (96) and 171
// (216) with k = 2.  Each XCD takes a contiguous eighth of the tiles, so that the
// halos of neighbours meet in one L2 (dealt out tile by tile: 512 float64 tubes 437,
// mixed 184, reading 1.47 and 0.93 of a read per step; 1600 cells 6.7).
// At most 221 registers, none spilled, because the two wavefronts' code is apart
// from the first load on (one body with branches spilled 136); held to three
// wavefronts per SIMD it spills 66 and takes half as long again.
// NG = 1 (float32): a wavefront holds whole cells and shares nothing; the
// second-order model's 66 values leave room for that.
//
// desc[0 .. ntubes): the tubes of this launch, steps = steps left before
// round 0, spin_limit = where the tube's status lies; first[k]: tube k's first
// tile.  Round `round` of the launches reads buffer (cur + round) & 1.
template <class M, class S, int NG>
__global__ void __launch_bounds__(64 * NG) __attribute__((amdgpu_waves_per_eu(2)))
k_tubes_tile(S *__restrict__ base, const TubeDesc *__restrict__ desc, const int *__restrict__ first, int ntubes,
             int tiles, int round, int ksteps, unsigned *__restrict__ status) {
  using D = Split<M, S, NG>;
  static_assert(D::CELLS == TUBE_TILE<S>);
  constexpr int T = TILE<S>;
  constexpr bool alone = NG == 1;
  static_assert(!alone || !D::halves);
  __shared__ Shared<M, S, NG> w;
  const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int cell = lane % D::CELLS, m = lane / D::CELLS; // m: which member (float64)
  const int sigma = 1 - 2 * m;
  const int tile = pair_block_order(blockIdx.x, gridDim.x);
  if (tile >= tiles) return;
  const int j = tube_of_tile(first, ntubes, tile);
  const TubeDesc d = desc[j];
  const int64_t left = d.steps - static_cast<int64_t>(round) * ksteps;
  const int k = left < ksteps ? static_cast<int>(left) : ksteps;
  if (k <= 0) return;
  const int cells = tube_tile_cells<S>(ksteps);
  const int h = MAXD * (k - 1);
  const int c0 = (tile - first[j]) * cells;
  const int n = d.n;
  int z = (c0 - h + cell) % n;
  if (z < 0) z += n;
  const bool store = cell >= h && cell < h + cells && c0 + cell - h < n;
  const int cur = (d.cur + round) & 1;
  const S *in = base + (cur ? d.off[1] : d.off[0]);
  S *out = base + (cur ? d.off[0] : d.off[1]);
  Relax rx;
  rx.mode = d.mode;
  rx.tau = d.tau;
  rx.eta_s = d.eta_s;
  int zo[2 * MAXD + 1];
#pragma unroll
  for (int s = -MAXD; s <= MAXD; ++s) {
    const int from = D::halves ? wrap_rt(z, sigma * s, n) : wrap_back(z, s, n);
    zo[s + MAXD] = static_cast<int>(tile_elem<M, S>(from)) + m * T;
  }
  // a wavefront runs its own group's code from here to the end; each passes the
  // same barriers
  for_group<NG>(grp, [&](auto G) {
    constexpr int q = decltype(G)::value;
    typename D::Pops f;
    D::template points<q>([&](auto I, auto P) {
      constexpr int i = decltype(I)::value;
      f[decltype(P)::value] = load_at(in + i * T, zo[M::P[i].tz + MAXD]);
    });
    __builtin_amdgcn_sched_barrier(0);
    unsigned flags = 0;
    for (int s = 0;; ++s) {
      const bool right = cell >= MAXD * s && cell < D::CELLS - MAXD * s;
      if constexpr (alone) {
        const Moments mo = moments<M>(f);
        Frame fr{1.0, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if (right) flags |= landau_frame(mo, fr);
        const double tau = relaxation_time<M>(rx, fr.n, fr.T);
        relax_cell<M, S>([&](auto I) { return f[decltype(I)::value]; }, fr, tau,
                         [&](auto I, S v) { f[decltype(I)::value] = v; });
      } else {
        // three barriers a step: the sums are written after the third and read
        // after the first, the frame after the first and read after the second and
        // third, rate and coefficients after the second and read after the third
        ShellSums mine[M::NSHELL]; // group 0
        shell_sums<D, M, q>(f, mine, w, lane);
        __syncthreads();
        if constexpr (q == 0) {
          const Moments mo = gathered_moments<D, M>(mine, w, lane);
          Frame fr{1.0, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
          if (right) flags |= landau_frame(mo, fr);
          share_frame(fr, w, cell);
        }
        __syncthreads();
        share_coefficients<D, M, S, q>(rx, w, cell);
        __syncthreads();
        relax_group<D, M, S, q>(f, w, lane);
      }
      if (s + 1 == k) break;
      int l = lane;
      asm volatile("" : "+v"(l));
      D::template points<q>([&](auto I, auto P) {
        constexpr int tz = M::P[decltype(I)::value].tz, p = decltype(P)::value;
        if constexpr (tz != 0) f[p] = from_lane(f[p], (l - sigma * tz) * 4);
      });
    }
    // fresh copies keep the compiler from forming every address before the loop
    int o = static_cast<int>(tile_elem<M, S>(z)) + m * T;
    int zero = 0;
    asm volatile("" : "+v"(o), "+s"(zero));
    S *dst = out + zero;
    if (store)
      D::template points<q>(
          [&](auto I, auto P) { store_plain(dst + decltype(I)::value * T, o, f[decltype(P)::value]); });
    if (flags) atomicOr(status + d.spin_limit, flags);
  });
}

} // namespace rlb
