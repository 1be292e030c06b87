// The time step with the populations of a cell split over the wavefronts of
// a workgroup, for tubes and small boxes.  A lane that holds a whole cell (or half of one)
// issues over 4000 instructions per step: 8-10 us at one wavefront per SIMD,
// however few cells there are.  Here the chain is cut:
//
// A workgroup of NG wavefronts works on 64 consecutive cells, one per lane.
// Each wavefront holds a part of the inversion pairs (Split) of all 64 cells:
// it gathers them, forms their part of the moments and, once the frame is
// known, relaxes and stores them.  The parts meet in LDS and every wavefront
// adds them up in the same order; the Landau solve and tau are computed by
// every wavefront for itself; the coefficients of the equilibrium are dealt
// out again (by parity block) and meet in LDS.  Two barriers per step.
#pragma once

#include "rlb_kernels.hpp"

namespace rlb {

// The inversion pairs of group g of NG.  float32: whole shells, so that the
// shells' sums are those of the one-lane kernels, bit for bit (NG = NSHELL,
// two groups of nearly equal size, or one of everything).  float64: NG runs of nearly equal
// size, whichever shells they meet, which share their part of the moments.
template <class M, class S, int NG>
struct Split {
  static constexpr bool by_shell = sizeof(S) == 4;
  static_assert(!by_shell || NG <= 2 || NG == M::NSHELL);
  static constexpr int owner(int l) { // the group of a shell
    constexpr int o3[4] = {0, 1, 1, 0}, o2[3] = {0, 0, 1};
    return NG == M::NSHELL ? l : NG == 1 ? 0 : M::ORDER == 3 ? o3[l] : o2[l];
  }
  static constexpr int begin(int g) { return M::Q / 2 * g / NG; } // float64
  // the pairs [seg_begin, seg_end) of group g in shell l
  static constexpr int seg_begin(int g, int l) {
    const int b = shell_pair_begin<M>(l);
    return by_shell || b > begin(g) ? b : begin(g);
  }
  static constexpr int seg_end(int g, int l) {
    const int e = shell_pair_begin<M>(l + 1);
    if (by_shell) return owner(l) == g ? e : seg_begin(g, l);
    return e < begin(g + 1) ? e : begin(g + 1);
  }
  static constexpr int size(int g, int l) {
    return seg_end(g, l) > seg_begin(g, l) ? seg_end(g, l) - seg_begin(g, l) : 0;
  }
  static constexpr int size(int g) {
    int n = 0;
    for (int l = 0; l < M::NSHELL; ++l) n += size(g, l);
    return n;
  }
  // place of pair k among the group's pairs
  static constexpr int local(int g, int k) {
    int n = 0;
    for (int l = 0; l < M::NSHELL; ++l) {
      if (size(g, l) && k >= seg_begin(g, l) && k < seg_end(g, l)) return n + k - seg_begin(g, l);
      n += size(g, l);
    }
    return -1;
  }
  static constexpr int max_size() {
    int m = 0;
    for (int g = 0; g < NG; ++g) m = size(g) > m ? size(g) : m;
    return m;
  }
  static constexpr int N = 2 * max_size();
  using Pops = S[N]; // the populations a lane holds: pair k at 2 local(k), 2 local(k) + 1
  // what is shared of the moments: the ShellSums of every shell, or every
  // group's part of the 14 moments
  static constexpr int SHARES = by_shell ? M::NSHELL : NG;
  static constexpr int SHARE = by_shell ? 10 : 14;

  // f(i, place) for the points of group G
  template <int G, class F>
  static __device__ __forceinline__ void points(F &&f) {
    static_for<0, M::NSHELL>([&](auto L) {
      constexpr int l = decltype(L)::value;
      if constexpr (size(G, l) > 0)
        static_for<2 * seg_begin(G, l), 2 * seg_end(G, l)>([&](auto I) {
          constexpr int i = decltype(I)::value;
          f(I, std::integral_constant<int, 2 * local(G, i / 2) + i % 2>{});
        });
    });
  }
};
static_assert(sizeof(ShellSums) == 10 * sizeof(double) && sizeof(Moments) == 14 * sizeof(double));

// What group G adds to the moments, left for the other wavefronts in `part`.
template <class D, class M, int G>
__device__ __forceinline__ void share_sums(const typename D::Pops &f, double (*part)[D::SHARE][64], int lane) {
  Moments m{};
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value;
    if constexpr (D::size(G, l) > 0) {
      ShellSums a{};
      static_for<D::seg_begin(G, l), D::seg_end(G, l)>([&](auto K) {
        constexpr int k = decltype(K)::value, p = D::local(G, k);
        const double x = static_cast<double>(f[2 * p]);
        const double y = static_cast<double>(f[2 * p + 1]);
        a.template add_pair<M, k>(x + y, x - y);
        a.pin();
      });
      if constexpr (D::by_shell) {
        const double *src = &a.sh;
#pragma unroll
        for (int j = 0; j < D::SHARE; ++j) part[l][j][lane] = src[j];
      } else {
        a.template fold<M, l>(m);
      }
    }
  });
  if constexpr (!D::by_shell) {
    const double *src = &m.N0;
#pragma unroll
    for (int j = 0; j < D::SHARE; ++j) part[G][j][lane] = src[j];
  }
}

// The moments of the lane's cell from all shares, in their order (after a
// barrier).
template <class D, class M>
__device__ __forceinline__ Moments gathered_moments(const double (*part)[D::SHARE][64], int lane) {
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
      for (int g = 1; g < D::SHARES; ++g) dst[j] += part[g][j][lane];
    }
  }
  return m;
}

// The wavefront that computes a parity block of the equilibrium's
// coefficients (blocks of 8, 5, 5, 5, 2, 2, 2 and 1, or 5, 2, 2, 2, 1, 1, 1).
template <class M, int NG>
constexpr int block_owner(int b) {
  constexpr int o3[8] = {0, 1, 2, 3, 1, 2, 3, 2}, o2[7] = {0, 1, 1, 2, 2, 2, 2};
  constexpr int h3[8] = {0, 1, 1, 1, 0, 0, 0, 0}, h2[7] = {0, 1, 1, 1, 0, 0, 0};
  if (NG == 2) return M::ORDER == 3 ? h3[b] : h2[b];
  return M::ORDER == 3 ? o3[b] : o2[b];
}

// The coefficients of group G's blocks in the theta-polynomials of every
// shell (eq_coefficients and shell_coefficients, operation for operation),
// left for all wavefronts in coef[shell][spatial part].
template <class M, class S, int NG, int G>
__device__ __forceinline__ void share_coefficients(const MJ &mj, S (*coef)[SpatialTable<M>::NS][64], int lane) {
  static_for<0, M::NBLOCK>([&](auto B) {
    constexpr int blk = decltype(B)::value;
    if constexpr (block_owner<M, NG>(blk) == G) {
      constexpr int b0 = M::BLOCK_BEGIN[blk], b1 = M::BLOCK_BEGIN[blk + 1];
      const EqBlock<M, blk> e = eq_block<M, blk>(mj);
      static_for<0, SpatialTable<M>::NS>([&](auto Sx) {
        constexpr int si = decltype(Sx)::value;
        if constexpr (spatial_block<M>(si) == blk) {
          static_for<0, M::NSHELL>([&](auto L) {
            constexpr int l = decltype(L)::value;
            coef[l][si][lane] = S(spatial_coefficient<M, l, si, b0, b1>(e.c));
          });
        }
      });
    }
  });
}

// Equilibrium and relaxation of the pairs of group G (relax_cell's
// arithmetic); post-collision values replace f.
template <class D, class M, class S, int G>
__device__ __forceinline__ void relax_group(typename D::Pops &f, const S (*coef)[SpatialTable<M>::NS][64], int lane,
                                            const Frame &fr, double tau) {
  using CT = S;
  const double g = fr.U0 / tau;
  const CT gg = CT(g);
  const CT bx = CT(g * fr.vx * M::INV_R), by = CT(g * fr.vy * M::INV_R), bz = CT(g * fr.vz * M::INV_R);
  static_for<0, M::NSHELL>([&](auto L) {
    constexpr int l = decltype(L)::value;
    if constexpr (D::size(G, l) > 0) {
      ShellCoef<M, CT> s;
#pragma unroll
      for (int si = 0; si < SpatialTable<M>::NS; ++si) s.c[si] = coef[l][si][lane];
      static_for<D::seg_begin(G, l), D::seg_end(G, l)>([&](auto K) {
        constexpr int k = decltype(K)::value, p = D::local(G, k);
        constexpr Point P = M::P[2 * k];
        CT E, O;
        shell_eval<M, 2 * k, CT>(s, E, O);
        const CT wE = CT(P.w) * E, wO = CT(P.w) * O;
        CT t = CT(0);
        if constexpr (P.tx != 0) t = fmadd(CT(P.tx), bx, t);
        if constexpr (P.ty != 0) t = fmadd(CT(P.ty), by, t);
        if constexpr (P.tz != 0) t = fmadd(CT(P.tz), bz, t);
        S &a = f[2 * p], &b = f[2 * p + 1];
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

// ---- one float64 step of a small box ------------------------------------------
//
// While the chip is not full a step lasts as long as a workgroup: the launch
// (3.8 us), the gathers' latency and one wavefront's chain, 1500 vector
// instructions here against 4300 in the two-lane kernel (k_step), which a
// larger box keeps hidden behind its memory traffic.  1 x 1 x 1600 10.7 -> 8.1
// us per step, 16^3 12.1 -> 9.8, 32^3 18.8 -> 14.4 (4.7 TB/s, from the caches).
// Offsets are 32-bit; the 24-bit multiply that forms them matters (32^3 16.5
// us with a 32-bit one).
template <class M, bool WALLS, int AC>
__global__ void __launch_bounds__(64 * M::NSHELL) __attribute__((amdgpu_waves_per_eu(2)))
k_step_split(InPtr<double, AC> cur, OutPtr<double, AC> nxt, Geom g, Relax rx, unsigned *__restrict__ status,
             const uint8_t *__restrict__ solid) {
  using S = double;
  constexpr int NG = M::NSHELL;
  using D = Split<M, S, NG>;
  constexpr int T = TILE<S>;
  __shared__ double part[D::SHARES][D::SHARE][64];
  __shared__ S coef[M::NSHELL][SpatialTable<M>::NS][64];
  const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  int cell = pair_block_order(blockIdx.x, gridDim.x) * 64 + lane;
  bool active = cell < g.cells;
  if (!active) cell = g.cells - 1; // computed, never stored
  if constexpr (WALLS) active = active && solid[cell] == 0;
  int x, y, z;
  cell_coords(cell, g, x, y, z);
  const Shifts sh(x, y, z, g);
  const uint32_t own = tile_bytes32<M, S>(cell);
  const char *in = reinterpret_cast<const char *>(cur);
  char *out = reinterpret_cast<char *>(nxt);
  constexpr int SEG = T * static_cast<int>(sizeof(S)); // bytes from a population to the next
  typename D::Pops f;
  for_group<NG>(grp, [&](auto G) {
    constexpr int q = decltype(G)::value;
    D::template points<q>([&](auto I, auto P) {
      constexpr int i = decltype(I)::value, p = decltype(P)::value;
      constexpr Point PT = M::P[i];
      const uint32_t o = AC == AA_EVEN ? own : tile_bytes32<M, S>(sh.template back<PT.tx, PT.ty, PT.tz>());
      f[p] = *reinterpret_cast<const S *>(in + (aa_odd(AC) ? i ^ 1 : i) * SEG + o);
    });
    __builtin_amdgcn_sched_barrier(0);
    share_sums<D, M, q>(f, part, lane);
  });
  __syncthreads();
  const Moments m = gathered_moments<D, M>(part, lane);
  Frame fr;
  const unsigned flags = landau_frame(m, fr);
  const double tau = relaxation_time<M>(rx, fr.n, fr.T);
  const MJ mj = mj_of(fr.n, fr.T, fr.U0, fr.Ux, fr.Uy, fr.Uz);
  for_group<NG>(grp, [&](auto G) { share_coefficients<M, S, NG, decltype(G)::value>(mj, coef, lane); });
  __syncthreads();
  for_group<NG>(grp, [&](auto G) {
    constexpr int q = decltype(G)::value;
    relax_group<D, M, S, q>(f, coef, lane, fr, tau);
    // AA_ODD: the offsets are formed again rather than kept through the
    // arithmetic (keeping them spills 112 registers: 64^3 119 instead of 111 us)
    int xs = x;
    asm volatile("" : "+v"(xs));
    const Shifts to(xs, y, z, g);
    if (active)
      D::template points<q>([&](auto I, auto P) {
        constexpr int i = decltype(I)::value, p = decltype(P)::value;
        constexpr Point PT = M::P[i];
        if constexpr (aa_odd(AC))
          *reinterpret_cast<S *>(out + i * SEG + tile_bytes32<M, S>(to.template fwd<PT.tx, PT.ty, PT.tz>())) = f[p];
        else
          __builtin_nontemporal_store(f[p], reinterpret_cast<S *>(out + (AC == AA_EVEN ? i ^ 1 : i) * SEG + own));
      });
  });
  if (active && flags && grp == 0) atomicOr(status, flags);
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
inline constexpr int TUBE_TILE = 64;
constexpr int tube_tile_cells(int k) { return TUBE_TILE - 2 * MAXD * (k - 1); }
inline constexpr int TUBE_MAX_KSTEPS = 5;
static_assert(tube_tile_cells(TUBE_MAX_KSTEPS) > 0);

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

// What bounds it.  Few tiles: the chain of one wavefront, 3.8-4.4 us per step
// (third order: 550 float64 instructions of the sum of the moments, the frame
// and tau, 550 of its own group, 110 of coefficients, two barriers).  A
// 1600-cell float64 tube takes 5.6 us per step with k = 5 (8.4 with k = 1; as
// one workgroup per tube, which uses one of 256 CUs, 74), mixed 5.1 (37).
// With more tiles than CUs, the arithmetic and the workgroups' turns at the
// barriers: 24 tubes of 200-4000 cells 22 us with k = 2 (196), mixed 16 (96);
// 512 of them 372 us (433), 2.9e9 updates/s.  float64 needs no more than 256
// registers, two wavefronts per SIMD, because the coefficients lie in LDS
// (with 30 of them in registers it spilled 200, and 512 tubes took 728 us).
// NG = 1 (float32): a wavefront holds whole cells and shares nothing; the
// second-order model's 66 values leave room for that.
//
// desc[0 .. ntubes): the tubes of this launch, steps = steps left before
// round 0, spin_limit = where the tube's status lies; first[k]: tube k's first
// tile.  Round `round` of the launches reads buffer (cur + round) & 1.
template <class M, class S, int NG>
__global__ void __launch_bounds__(64 * NG) __attribute__((amdgpu_waves_per_eu(2)))
k_tubes_tile(S *__restrict__ base, const TubeDesc *__restrict__ desc, const int *__restrict__ first, int ntubes,
             int round, int ksteps, unsigned *__restrict__ status) {
  using D = Split<M, S, NG>;
  constexpr int T = TILE<S>;
  constexpr bool alone = NG == 1;
  __shared__ double part[alone ? 1 : D::SHARES][D::SHARE][64];
  __shared__ S coef[alone ? 1 : M::NSHELL][SpatialTable<M>::NS][64];
  const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int tile = static_cast<int>(blockIdx.x);
  const int j = tube_of_tile(first, ntubes, tile);
  const TubeDesc d = desc[j];
  const int64_t left = d.steps - static_cast<int64_t>(round) * ksteps;
  const int k = left < ksteps ? static_cast<int>(left) : ksteps;
  if (k <= 0) return;
  const int cells = tube_tile_cells(ksteps);
  const int h = MAXD * (k - 1);
  const int c0 = (tile - first[j]) * cells;
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
    D::template points<q>([&](auto I, auto P) {
      constexpr int i = decltype(I)::value;
      f[decltype(P)::value] = load_at(in + i * T, zo[M::P[i].tz + MAXD]);
    });
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!alone) share_sums<D, M, q>(f, part, lane);
  });
  unsigned flags = 0;
  for (int s = 0;; ++s) {
    // two barriers a step: part is written after the second and read after
    // the first, coef the other way round
    Moments m;
    if constexpr (alone) {
      m = moments<M>(f);
    } else {
      __syncthreads();
      m = gathered_moments<D, M>(part, lane);
    }
    Frame fr{1.0, 1.0, 1.0, 1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (lane >= MAXD * s && lane < TUBE_TILE - MAXD * s) flags |= landau_frame(m, fr);
    const double tau = relaxation_time<M>(rx, fr.n, fr.T);
    if constexpr (alone) {
      relax_cell<M, S>([&](auto I) { return f[decltype(I)::value]; }, fr, tau,
                       [&](auto I, S v) { f[decltype(I)::value] = v; });
    } else {
      const MJ mj = mj_of(fr.n, fr.T, fr.U0, fr.Ux, fr.Uy, fr.Uz);
      for_group<NG>(grp, [&](auto G) { share_coefficients<M, S, NG, decltype(G)::value>(mj, coef, lane); });
      __syncthreads();
    }
    const bool last = s + 1 == k;
    for_group<NG>(grp, [&](auto G) {
      constexpr int q = decltype(G)::value;
      if constexpr (!alone) relax_group<D, M, S, q>(f, coef, lane, fr, tau);
      if (last) {
        // fresh copies keep the compiler from forming every address before the loop
        int o = static_cast<int>(tile_elem<M, S>(z));
        int zero = 0;
        asm volatile("" : "+v"(o), "+s"(zero));
        S *dst = out + zero;
        if (store)
          D::template points<q>(
              [&](auto I, auto P) { store_plain(dst + decltype(I)::value * T, o, f[decltype(P)::value]); });
      } else {
        int l = lane;
        asm volatile("" : "+v"(l));
        D::template points<q>([&](auto I, auto P) {
          constexpr int tz = M::P[decltype(I)::value].tz, p = decltype(P)::value;
          if constexpr (tz != 0) f[p] = from_lane(f[p], (l - tz) * 4);
        });
        if constexpr (!alone) share_sums<D, M, q>(f, part, lane);
      }
    });
    if (last) break;
  }
  if (flags && grp == 0) atomicOr(status + d.spin_limit, flags);
}

} // namespace rlb
