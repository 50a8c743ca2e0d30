// Host-side launch entry points, and the choice of a step's instance from its arguments
// (launch_one, instantiated per lattice, precision and number of scalars in generated units).
#pragma once

#include "lbm_step.hpp"

namespace lbm {

// LAUNCH_STEP: every cell in one instance (FULL with curved walls, observables or mixture
// transport); LAUNCH_STEP_SPLIT (D2Q9): a.nlb blocks of listed boundary cells and nblocks
// tiles of interior cells in one launch; LAUNCH_STEP_INTERIOR / LAUNCH_STEP_LIST (D3Q27): the
// two halves of a split step (interior cells, FULL with mixture transport; then the listed
// boundary cells, FULL with curved walls or mixture transport).
enum LaunchKind {
  LAUNCH_STEP = 0, LAUNCH_EXTRACT = 1, LAUNCH_INIT = 2, LAUNCH_STEP_INTERIOR = 3, LAUNCH_STEP_LIST = 4,
  LAUNCH_STEP_SPLIT = 5
};

// Returns hipSuccess or the launch error.  nblocks covers N cells with 256 threads.
hipError_t launch_d2q9(int prec, int ns, int kind, const StepArgs &a, int nblocks, hipStream_t st,
                       const double *Ph, const double *u, const double *scal);
hipError_t launch_d3q27(int prec, int ns, int kind, const StepArgs &a, int nblocks, hipStream_t st,
                        const double *Ph, const double *u, const double *scal);
hipError_t launch_geometry(int Q, const uint8_t *solid, void *geom, int nx, int ny, int nz, long long N,
                           const int *face, hipStream_t st);
hipError_t launch_geometry_levelset(int Q, const double *phi, void *geom, int nx, int ny, int nz, long long N,
                                    const int *face, hipStream_t st);
// Adjoint launches (lbm_adjoint.hip).  kind 0: reverse step (p0 lamB, p1 lamT', p2 lamA out,
// p3 lamT out, p4 coefficient scratch); 1/2: objective sums / gradient (p2 lamA, p3 lamT);
// 3: reverse of the initialisation (p0 lamA, p1 lamT, u0, gu out, p3 grad T out).
hipError_t launch_adjoint(int prec, int ns, int kind, const StepArgs &sa, int nblocks, hipStream_t st, const void *p0,
                          const void *p1, void *p2, void *p3, void *p4, double mean_T, const double *u0, double *gu);
// Sums of the per-block records into out[NSUM] and, with a host copy of the work buffer's
// head (out is then its sums), the head to the host.
hipError_t launch_finalize(const double *partials, int nrec, double *stage, double *out, hipStream_t st,
                           const double *head = nullptr, double *host = nullptr);
hipError_t launch_finalize_one(const double *partials, int nrec, double *stage, double *out, hipStream_t st,
                               const double *head = nullptr, double *host = nullptr);   // one counter per record
hipError_t launch_publish(const double *head, double *host, hipStream_t st);   // nothing without a host copy
// Two arrays (bytes multiples of 16, 16-byte aligned) copied in one launch, and the head.
hipError_t launch_copy_state(const void *a, void *da, size_t abytes, const void *b, void *db, size_t bbytes,
                             const double *head, double *host, hipStream_t st);
hipError_t launch_set_thermo(double *thermo, double pi, double q, double K, hipStream_t st);
// Closed domain: (pi, q, K) of the next level from the step's nrec block records.
hipError_t launch_thermo(const double *partials, int nrec, double *thermo, hipStream_t st);
// Observables: flame-surface block records (one double each) and mean / RMS fields.
hipError_t launch_surface(int Q, int prec, const StepArgs &a, int nblocks, hipStream_t st, double T_u, double T_b);
hipError_t launch_statistics(const double *acc, int D, long long N, long long k, double P0, double *mean, double *rms,
                             hipStream_t st);

// Collision instance for the parameters: BGK, or the cumulant operator with every order
// >= 3 at rate one (decided in the compute precision, as the kernel would), or general
// (other rates, or the parameterised higher orders, a runtime switch of that instance).
template <int Q, int PREC>
int collision_instance(const StepArgs &a) {
  using R = typename Prec<PREC>::R;
  if (a.collision != 0) return COLL_BGK;
  return (Q == 27 && ((R)a.wh != R(1) || a.p4)) ? COLL_CUM : COLL_CUM1;
}

// Every face periodic and no solid cell: no cell needs boundary code.
inline bool without_boundaries(const StepArgs &a) {
  bool free = !a.geom;
  for (int f = 0; f < 6; ++f) free = free && a.face[f] < 0;
  return free;
}

template <int Q, int PREC, int NS, bool FULL, int MODE>
hipError_t launch_step(const StepArgs &a, int nblocks, hipStream_t st) {
  using R = typename Prec<PREC>::R;
  switch (collision_instance<Q, PREC>(a)) {
    case COLL_CUM1: {
      constexpr bool free = MODE == MODE_FREE || MODE == MODE_FREE_LIN;
      constexpr bool inter = MODE == MODE_INTERIOR || MODE == MODE_INTERIOR_LIN;
      // FP32 steps without boundaries: dynamic LDS beside the 18432 B of the block sums leaves four
      // blocks a CU (160 KiB of LDS, given out in units of 1280 B) instead of up to eight.  More waves in
      // flight than the memory side needs cost it locality: HIT, us per step at 8 / 7 / 6 / 5 / 4 / 3
      // blocks, 256^3 667 / 663 / 656 / 650 / 649 / 655, 512x128x512 1348 / 1350 / 1340 / 1322 / 1316 /
      // 1362; at 8 / 5 / 4, 128^3 88.0 / 85.8 / 85.7, 300^3 1159 / 1154 / 1148, passive 256x256x512 1421 /
      // 1409 / 1376.  From 4096 tiles: 2304 26.3 / 26.3 / 26.9, 3072 37.9 / 36.8 / 37.6, 4096 44.7 / 43.4 /
      // 43.7.  Of some fifty grids above the line a few lost, by 0.3 to 1.2 % (passive 128^3 91.3 / 91.2 /
      // 92.4, HIT 224^3 485 / 489 / 489); 512x256x256 gained or lost 4 % (1368 / 1322 / 1313, 1333 / 1359 /
      // 1384) with the place of its buffers.  FP16 storage, bound by issue, wants all its waves (HIT
      // 256^3 377 / 396 / 422).
      const unsigned lds = Q == 27 && PREC == 1 && free && nblocks >= 4096 ? 14000 : 0;
      // SEG by kind of step, not by size, so that a grid rounds as its copies side by side do
      constexpr bool seg = Q == 27 && ((PREC != 0 && NS == 6 && inter) || (PREC == 2 && free)) && !FULL;
      // The plain instances also come with cached pull loads (large grids): the interior ones, and
      // with fewer than two scalars those of every cell (more scalars split on such grids), but
      // for the boundary-free FP64 one of D3Q27, which serves small grids.
      constexpr bool cached = !FULL && MODE != MODE_LIST && (inter || NS < 2) && !(free && Q == 27 && PREC == 0);
      auto run = [&](auto pullc, auto segment) {
        hipLaunchKernelGGL((step_kernel<Q, PREC, NS, false, FULL, COLL_CUM1, MODE, decltype(pullc)::value,
                                        decltype(segment)::value>), dim3(nblocks), dim3(256), lds, st, to_kargs<R>(a));
      };
      auto run_pull = [&](auto segment) {
        if constexpr (cached) {
          if (a.pull_cached) return run(std::true_type{}, segment);
        }
        run(std::false_type{}, segment);
      };
      if constexpr (seg && free) {                     // never with curved walls
        run_pull(std::true_type{});
      } else if constexpr (seg) {
        if (a.lvl) run_pull(std::false_type{});
        else run_pull(std::true_type{});
      } else {
        run_pull(std::false_type{});
      }
      break;
    }
    case COLL_CUM:
      if constexpr (Q == 27)
        hipLaunchKernelGGL((step_kernel<Q, PREC, NS, false, FULL, COLL_CUM, MODE>), dim3(nblocks), dim3(256), 0, st,
                           to_kargs<R>(a));
      else
        return hipErrorInvalidValue;
      break;
    default:
      hipLaunchKernelGGL((step_kernel<Q, PREC, NS, false, FULL, COLL_BGK, MODE>), dim3(nblocks), dim3(256), 0, st,
                         to_kargs<R>(a));
  }
  return hipGetLastError();
}

template <int PREC, int NS, bool LFULL, bool IFULL, int IMODE>
hipError_t launch_split(const StepArgs &a, int nblocks, hipStream_t st) {
  using R = typename Prec<PREC>::R;
  const dim3 grid(nblocks + a.nlb), block(256);
  if (collision_instance<9, PREC>(a) == COLL_BGK)
    hipLaunchKernelGGL((split_kernel<PREC, NS, LFULL, IFULL, COLL_BGK, IMODE, false>), grid, block, 0, st, to_kargs<R>(a));
  else if (!IFULL && a.pull_cached)
    hipLaunchKernelGGL((split_kernel<PREC, NS, LFULL, IFULL, COLL_CUM1, IMODE, !IFULL>), grid, block, 0, st,
                       to_kargs<R>(a));
  else
    hipLaunchKernelGGL((split_kernel<PREC, NS, LFULL, IFULL, COLL_CUM1, IMODE, false>), grid, block, 0, st,
                       to_kargs<R>(a));
  return hipGetLastError();
}

// The instances of a split step: the list FULL with curved walls, observables or mixture
// transport, the tiles with the latter two.  Fewer than two scalars split for curved walls alone.
template <int PREC, int NS, int IMODE>
hipError_t launch_split_kind(const StepArgs &a, int nblocks, hipStream_t st) {
  if (a.stats || a.probe_out || a.mix) return launch_split<PREC, NS, true, true, IMODE>(a, nblocks, st);
  if constexpr (NS >= 2) {
    if (!a.lvl) return launch_split<PREC, NS, false, false, IMODE>(a, nblocks, st);
  }
  return launch_split<PREC, NS, true, false, IMODE>(a, nblocks, st);
}

template <int Q, int PREC, int NS>
hipError_t launch_one(int kind, const StepArgs &a, int nblocks, hipStream_t st, const double *Ph,
                      const double *u, const double *scal) {
  using R = typename Prec<PREC>::R;
  const bool full = a.lvl || a.stats || a.probe_out || a.mix;
  switch (kind) {
    case LAUNCH_STEP:
      if (full) return launch_step<Q, PREC, NS, true, MODE_ALL>(a, nblocks, st);
      // No boundary anywhere: no boundary code (us per step, all-cell / free instance: vortex
      // 128^2 FP64 6.0 / 4.8, HIT 100^3 FP16 storage 28.2 / 27.4, 32^3 FP32 6.6 / 5.9, two-step 64^3 FP64
      // 48 / 38).  D3Q27 in FP64: not with one scalar (48^3 12.3 / 12.8, 128^3 181 / 182, 256x256x192
      // 1068 / 1059), and isothermal up to 4096 tiles (32^3 7.9 / 7.2, 64^3 24.8 / 24.3, 128x64x96 71.4 /
      // 71.0, 128x128x64 87.6 / 88.0; 125^3 192.0 / 194.1, 192^3 597 / 600, 250^3 1368 / 1386, 256^3 1327 /
      // 1332, and no better with fewer resident blocks: 125^3 195, 192^3 602, 250^3 1384, 256^3 1321).
      if constexpr (!(Q == 27 && PREC == 0 && NS == 1)) {
        if (without_boundaries(a) && (Q != 27 || PREC != 0 || nblocks <= 4096))
          return a.band_rows ? launch_step<Q, PREC, NS, false, MODE_FREE>(a, nblocks, st)
                             : launch_step<Q, PREC, NS, false, MODE_FREE_LIN>(a, nblocks, st);
      }
      return launch_step<Q, PREC, NS, false, MODE_ALL>(a, nblocks, st);
    case LAUNCH_STEP_SPLIT:      // interior cells FULL with observables or mixture transport
      if constexpr (Q == 9)
        return a.band_rows ? launch_split_kind<PREC, NS, MODE_INTERIOR>(a, nblocks, st)
                           : launch_split_kind<PREC, NS, MODE_INTERIOR_LIN>(a, nblocks, st);
      return hipErrorInvalidValue;
    case LAUNCH_STEP_INTERIOR:   // on the 64x4 tile grid when it fits, else on linear tiles
      if constexpr (Q == 27) {
        if constexpr (NS == 6) {
          if (a.mix)
            return a.band_rows ? launch_step<Q, PREC, NS, true, MODE_INTERIOR>(a, nblocks, st)
                               : launch_step<Q, PREC, NS, true, MODE_INTERIOR_LIN>(a, nblocks, st);
        }
        return a.band_rows ? launch_step<Q, PREC, NS, false, MODE_INTERIOR>(a, nblocks, st)
                           : launch_step<Q, PREC, NS, false, MODE_INTERIOR_LIN>(a, nblocks, st);
      }
      return hipErrorInvalidValue;
    case LAUNCH_STEP_LIST:       // plain only with two scalars or more: the others split for curved walls alone
      if constexpr (Q == 27) {
        if constexpr (NS >= 2) {
          if (!a.lvl && !a.mix) return launch_step<Q, PREC, NS, false, MODE_LIST>(a, nblocks, st);
        }
        return launch_step<Q, PREC, NS, true, MODE_LIST>(a, nblocks, st);
      }
      return hipErrorInvalidValue;
    case LAUNCH_EXTRACT:   // no collision on the extract path
      if (full)
        hipLaunchKernelGGL((step_kernel<Q, PREC, NS, true, true, COLL_CUM1, MODE_ALL>), dim3(nblocks), dim3(256), 0,
                           st, to_kargs<R>(a));
      else
        hipLaunchKernelGGL((step_kernel<Q, PREC, NS, true, false, COLL_CUM1, MODE_ALL>), dim3(nblocks), dim3(256), 0,
                           st, to_kargs<R>(a));
      break;
    default:
      hipLaunchKernelGGL((init_kernel<Q, PREC, NS>), dim3(nblocks), dim3(256), 0, st, to_kargs<double>(a), Ph, u,
                         scal, const_cast<double *>(a.thermo));
  }
  return hipGetLastError();
}

template <int Q, int PREC>
hipError_t launch_ns(int ns, int kind, const StepArgs &a, int nblocks, hipStream_t st, const double *Ph,
                     const double *u, const double *scal) {
  switch (ns) {
    case 0: return launch_one<Q, PREC, 0>(kind, a, nblocks, st, Ph, u, scal);
    case 1: return launch_one<Q, PREC, 1>(kind, a, nblocks, st, Ph, u, scal);
    case 2: return launch_one<Q, PREC, 2>(kind, a, nblocks, st, Ph, u, scal);
    case 6: return launch_one<Q, PREC, 6>(kind, a, nblocks, st, Ph, u, scal);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
