// D2Q9 dispatch over precisions and scalar counts (the instances are generated units, one per
// precision and number of scalars), and the launches of the kernels that both lattices share.
#include "lbm_launch.hpp"

namespace lbm {
hipError_t launch_d2q9(int prec, int ns, int kind, const StepArgs &a, int nblocks, hipStream_t st,
                       const double *Ph, const double *u, const double *scal) {
  switch (prec) {
    case 0: return launch_ns<9, 0>(ns, kind, a, nblocks, st, Ph, u, scal);
    case 1: return launch_ns<9, 1>(ns, kind, a, nblocks, st, Ph, u, scal);
    case 2: return launch_ns<9, 2>(ns, kind, a, nblocks, st, Ph, u, scal);
  }
  return hipErrorInvalidValue;
}

template <class Src>
static hipError_t geometry(int Q, const Src *solid, void *geom, int nx, int ny, int nz, long long N, const int *f,
                           hipStream_t st) {
  const int nb = (int)((N + 255) / 256);
  if (Q == 9)
    hipLaunchKernelGGL((geometry_kernel<9, Src>), dim3(nb), dim3(256), 0, st, solid, geom, nx, ny, nz, N, f[0],
                       f[1], f[2], f[3], f[4], f[5]);
  else
    hipLaunchKernelGGL((geometry_kernel<27, Src>), dim3(nb), dim3(256), 0, st, solid, geom, nx, ny, nz, N, f[0],
                       f[1], f[2], f[3], f[4], f[5]);
  return hipGetLastError();
}

hipError_t launch_geometry(int Q, const uint8_t *solid, void *geom, int nx, int ny, int nz, long long N,
                           const int *f, hipStream_t st) {
  return geometry(Q, solid, geom, nx, ny, nz, N, f, st);
}

hipError_t launch_geometry_levelset(int Q, const double *phi, void *geom, int nx, int ny, int nz, long long N,
                                    const int *f, hipStream_t st) {
  return geometry(Q, phi, geom, nx, ny, nz, N, f, st);
}

template <int W>
static hipError_t reduce(const double *rec, int nrec, double *stage, double *out, hipStream_t st, const double *head,
                         double *host) {
  // one launch up to 4096 records; more in chunks of at least 512 (at most 256 of them) first
  if (nrec > 4096) {
    const int chunk = nrec > 512 * 256 ? (nrec + 255) / 256 : 512;
    const int nb = (nrec + chunk - 1) / chunk;
    hipLaunchKernelGGL(reduce_records<W>, dim3(nb), dim3(1024), 0, st, rec, nrec, chunk, stage, (const double *)nullptr,
                       (double *)nullptr);
    rec = stage;
    nrec = nb;
  }
  hipLaunchKernelGGL(reduce_records<W>, dim3(1), dim3(1024), 0, st, rec, nrec, nrec, out, head, host);
  return hipGetLastError();
}

hipError_t launch_finalize(const double *partials, int nrec, double *stage, double *out, hipStream_t st,
                           const double *head, double *host) {
  return reduce<NSUM>(partials, nrec, stage, out, st, head, host);
}

hipError_t launch_finalize_one(const double *partials, int nrec, double *stage, double *out, hipStream_t st,
                               const double *head, double *host) {
  return reduce<1>(partials, nrec, stage, out, st, head, host);
}

hipError_t launch_publish(const double *head, double *host, hipStream_t st) {
  if (!host) return hipSuccess;
  hipLaunchKernelGGL(publish_kernel, dim3(1), dim3(64), 0, st, head, host);
  return hipGetLastError();
}

hipError_t launch_copy_state(const void *a, void *da, size_t abytes, const void *b, void *db, size_t bbytes,
                             const double *head, double *host, hipStream_t st) {
  const size_t na = abytes / 16, nb = bbytes / 16, most = na > nb ? na : nb;
  const size_t blocks = (most + 1023) / 1024;
  const dim3 grid((unsigned)(blocks < 1 ? 1 : blocks > 16384 ? 16384 : blocks));
  if (abytes + bbytes > ((size_t)128 << 20))      // source and destination exceed the Infinity Cache
    hipLaunchKernelGGL(copy_state_kernel<true>, grid, dim3(256), 0, st, (const u32x4 *)a, (u32x4 *)da, na, (const u32x4 *)b,
                       (u32x4 *)db, nb, head, host);
  else
    hipLaunchKernelGGL(copy_state_kernel<false>, grid, dim3(256), 0, st, (const u32x4 *)a, (u32x4 *)da, na, (const u32x4 *)b,
                       (u32x4 *)db, nb, head, host);
  return hipGetLastError();
}

hipError_t launch_thermo(const double *partials, int nrec, double *thermo, hipStream_t st) {
  hipLaunchKernelGGL(thermo_kernel, dim3(1), dim3(1024), 0, st, partials, nrec, thermo);
  return hipGetLastError();
}

hipError_t launch_surface(int Q, int prec, const StepArgs &a, int nblocks, hipStream_t st, double T_u, double T_b) {
  const KArgs<double> k = to_kargs<double>(a);
  const double inv = 1.0 / (T_b - T_u);
  if (Q == 9) {
    if (prec == 0) hipLaunchKernelGGL((surface_kernel<9, 0>), dim3(nblocks), dim3(256), 0, st, k, inv);
    else hipLaunchKernelGGL((surface_kernel<9, 1>), dim3(nblocks), dim3(256), 0, st, k, inv);
  } else {
    if (prec == 0) hipLaunchKernelGGL((surface_kernel<27, 0>), dim3(nblocks), dim3(256), 0, st, k, inv);
    else hipLaunchKernelGGL((surface_kernel<27, 1>), dim3(nblocks), dim3(256), 0, st, k, inv);
  }
  return hipGetLastError();
}

hipError_t launch_statistics(const double *acc, int D, long long N, long long k, double P0, double *mean, double *rms,
                             hipStream_t st) {
  const int nb = (int)((N + 255) / 256);
  hipLaunchKernelGGL(statistics_kernel, dim3(nb), dim3(256), 0, st, acc, D, N, (double)k, P0, mean, rms);
  return hipGetLastError();
}

hipError_t launch_set_thermo(double *thermo, double pi, double q, double K, hipStream_t st) {
  hipLaunchKernelGGL(set_thermo_kernel, dim3(1), dim3(64), 0, st, thermo, pi, q, K);
  return hipGetLastError();
}
}  // namespace lbm
