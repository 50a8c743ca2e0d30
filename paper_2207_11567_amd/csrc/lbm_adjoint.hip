// Adjoint kernels and their C entry points (include/lbm.h, differentiation section):
// one reverse step of the fused LB/FD step, the objective J = sum rho |u|^2 / 2 +
// sum (T - mean T)^2 with its gradient with respect to the state, and the reverse of the
// equilibrium initialisation.  Scope: D3Q27, periodic faces, no solids, isothermal or
// passive temperature, cumulant collision with every order >= 3 at rate one; FP64 or FP32.
#include <math.h>
#include <string.h>

#include <string>

#include "../../include/lbm.h"
#include "lbm_adjoint.hpp"

namespace lbm {

// Cell of this thread (256 consecutive ones per block, each XCD on a contiguous part of the
// grid) and the offsets of its periodic neighbours at -2..2 on each axis.
template <class A> __device__ __forceinline__ int adjoint_cell(const A &a, int (&off)[3][5]) {
  const int nxy = a.nx * a.ny;
  const int n = tile_of_block(blockIdx.x, gridDim.x, a.remap) * 256 + (int)threadIdx.x;
  const int z = n / nxy, rem = n - z * nxy, y = rem / a.nx, x = rem - y * a.nx;
  int code[5];
  axis_offsets(x, a.nx, -1, -1, 1, off[0], code);
  axis_offsets(y, a.ny, -1, -1, a.nx, off[1], code);
  axis_offsets(z, a.nz, -1, -1, nxy, off[2], code);
  return n;
}
// Index of the cell at -c_i.
__device__ __forceinline__ unsigned adjoint_source(unsigned un, int i, const int (&off)[3][5]) {
  return un + (unsigned)(off[0][2 - cx(i)] + off[1][2 - cy(i)] + off[2][2 - cz(i)]);
}

// One reverse step of a cell.  Bound by memory: the populations, their adjoint in and out, and
// the 13 coefficients of the scalar (440 B per FP32 cell) at two waves per SIMD in FP32 (three
// 27-vectors live; asked for three waves it spills and takes 225 us) and one in FP64.  The pull
// takes raw buffer loads with shared 32-bit offsets, everything after it plain accesses: as
// buffer ones the loads could not pass the stores of the coefficients, and the axes waited for
// one another.  The stencil's neighbours: in FP32 all four of each axis, loaded before the velocity
// is known; in FP64, where registers are short, the three upwind ones.  NT streams the incoming
// adjoint, which is read once (FP32 where the step's arrays exceed the Infinity Cache, below).
// us per step, global loads in linear order / this: FP32 passive 128^3 195 / 186 (5.0 TB/s), 100x90x110
// 99 / 87, 64^3 26.0 / 25.5, 48^3 14.8 / 13.4, isothermal 128^3 145 / 139, 64^3 18.7 / 18.2; FP64 passive 128^3
// 427 / 422, 128x96x96 233 / 236, 64^3 46.5 / 46.9, 48^3 26.1 / 25.7, 24^3 12.0 / 12.0.  On the step's 64x4
// tiles with scalar y and z the FP32 passive one took 204 at 128^3.
template <int PREC, int NS, bool NT>
__global__ __launch_bounds__(256) void adjoint_kernel(KArgs<typename Prec<PREC>::R> a,
                    const typename Prec<PREC>::R *__restrict__ lamB,
                    const typename Prec<PREC>::R *__restrict__ lamT1, typename Prec<PREC>::R *__restrict__ lamA,
                    typename Prec<PREC>::R *__restrict__ coef) {
  using P = Prec<PREC>;
  using St = typename P::St;
  using R = typename P::R;
  using Sc = typename P::Sc;
  constexpr R s = R(1.0 / 3.0);
  const int N = a.N;
  int off[3][5];
  const int n = adjoint_cell(a, off);
  if (n >= N) return;
  const unsigned un = (unsigned)n;
  const St *__restrict__ pin = (const St *)a.pop_in;
  const Sc *__restrict__ T = (const Sc *)a.scal_in;
  // pull (forward recompute)
  R g[27];
#pragma unroll
  for (int i = 0; i < 27; ++i) g[i] = decode<R>(bld<St>(slice(pin + (size_t)i * N), adjoint_source(un, i, off)));
  R nb[3][4];                                       // the scalar at -2, -1, +1, +2 per axis
  if constexpr (NS == 1 && PREC != 0) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 4; ++k) nb[d][k] = (R)ldg(T, un + (unsigned)off[d][k < 2 ? k : k + 1]);
  }
  const R rho0 = a.th.rho_ref;
  const R mom = fdiv(a.P0, s * rho0);
  R mx = R(0), my = R(0), mz = R(0);
#pragma unroll
  for (int i = 0; i < 27; ++i) {
    if (cx(i)) mx += R(cx(i)) * g[i];
    if (cy(i)) my += R(cy(i)) * g[i];
    if (cz(i)) mz += R(cz(i)) * g[i];
  }
  const R u[3] = {mx * mom, my * mom, mz * mom};
  R lu[3] = {R(0), R(0), R(0)};
  if constexpr (NS == 1) {
    // T' = T + K lap T - sum_d |u_d| W_d: adjoint of the advection part, per axis
    const R T0 = (R)ldg(T, un);
    const R lT = lamT1[n];
    R self = R(0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const bool up = u[d] >= R(0);
      R U1, D1, U2;                                 // the upwind-ordered neighbours of the stencil
      if constexpr (PREC != 0) {
        U1 = up ? nb[d][1] : nb[d][2];
        D1 = up ? nb[d][2] : nb[d][1];
        U2 = up ? nb[d][0] : nb[d][3];
      } else {
        U1 = (R)ldg(T, un + (unsigned)(up ? off[d][1] : off[d][3]));
        D1 = (R)ldg(T, un + (unsigned)(up ? off[d][3] : off[d][1]));
        U2 = (R)ldg(T, un + (unsigned)(up ? off[d][0] : off[d][4]));
      }
      R dW[4];
      const R W = weno3_diff_grad(U2, U1, T0, D1, a.eps[0], dW);
      lu[d] += up ? -lT * W : lT * W;               // d(-|u| W)/du = -sign(u) W
      const R c = -lT * fabs(u[d]);
      // contributions to the positions -2, -1, +1, +2 along d (and to the cell itself)
      const R cU2 = c * dW[0], cU1 = c * dW[1], cD1 = c * dW[3];
      coef[(size_t)(4 * d + 0) * N + n] = up ? cU2 : R(0);
      coef[(size_t)(4 * d + 1) * N + n] = up ? cU1 : cD1;
      coef[(size_t)(4 * d + 2) * N + n] = up ? cD1 : cU1;
      coef[(size_t)(4 * d + 3) * N + n] = up ? R(0) : cU2;
      self += c * dW[2];
    }
    coef[(size_t)12 * N + n] = self;
  }
  // collision reverse pass
  R lam[27];
#pragma unroll
  for (int i = 0; i < 27; ++i)
    lam[i] = NT ? __builtin_nontemporal_load(lamB + (size_t)i * N + n) : lamB[(size_t)i * N + n];
  Rates<R> rt;
  rt.tau0 = viscosity(a.th, rho0) * R(3) + R(0.5);
  rt.smag18 = a.smag18;
  rt.wb = a.wb;
  rt.wh = a.wh;
  rt.gal = false;
  rt.p4 = false;
  collide_d3q27_vjp(g, mom, rt, lam, lu);
  // transposed streaming: the adjoint of g_i(r) = A_i(r - c_i) is pushed to r - c_i
#pragma unroll
  for (int i = 0; i < 27; ++i) stg(lamA + (size_t)i * N, adjoint_source(un, i, off), lam[i]);
}

// lamT(s) = lamT'(s) + K lap(lamT')(s) + self(s) + gathered advection contributions.
template <int PREC>
__global__ __launch_bounds__(256) void adjoint_scalar_kernel(KArgs<typename Prec<PREC>::R> a,
                                                             const typename Prec<PREC>::R *__restrict__ lamT1,
                                                             const typename Prec<PREC>::R *__restrict__ coef,
                                                             typename Prec<PREC>::R *__restrict__ lamT) {
  using R = typename Prec<PREC>::R;
  const int N = a.N;
  int off[3][5];
  const int n = adjoint_cell(a, off);
  if (n >= N) return;
  const unsigned un = (unsigned)n;
  const R rho0 = a.th.rho_ref;
  const R rhoD0 = rho0 * viscosity(a.th, rho0) * a.th.inv_Pr;
  const R K = fdiv(a.th.F, rho0) * rhoD0;
  const auto sl = slice(lamT1);
  const R l0 = bld<R>(sl, un);
  R lap = R(0), acc = bld<R>(slice(coef + (size_t)12 * N), un);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lap += bld<R>(sl, un + (unsigned)off[d][3]) + bld<R>(sl, un + (unsigned)off[d][1]) - R(2) * l0;
    auto from = [&](int j, int k) { return bld<R>(slice(coef + (size_t)(4 * d + j) * N), un + (unsigned)off[d][k]); };
    acc += from(0, 4);      // from the cell at +2 (its -2 slot)
    acc += from(1, 3);      // from +1 (its -1 slot)
    acc += from(2, 1);      // from -1 (its +1 slot)
    acc += from(3, 0);      // from -2 (its +2 slot)
  }
  bst<R>(slice(lamT), un, l0 + K * lap + acc);
}

// Objective pieces at the state: block records of (rho|u|^2/2, T, T^2).
template <int PREC, int NS>
__global__ __launch_bounds__(256) void objective_kernel(KArgs<typename Prec<PREC>::R> a, double mean_T, int pass,
                                                        typename Prec<PREC>::R *__restrict__ lamA,
                                                        typename Prec<PREC>::R *__restrict__ lamT) {
  using P = Prec<PREC>;
  using St = typename P::St;
  using R = typename P::R;
  using Sc = typename P::Sc;
  constexpr R s = R(1.0 / 3.0);
  const int n = blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
  const int N = a.N;
  double red[NSUM];
#pragma unroll
  for (int k = 0; k < NSUM; ++k) red[k] = 0.0;
  if (n < N) {
    const unsigned un = (unsigned)n;
    const St *__restrict__ pin = (const St *)a.pop_in;
    const int nxy = a.nx * a.ny;
    const int z = n / nxy, rem = n - z * nxy, y = rem / a.nx, x = rem - y * a.nx;
    const AxisNb ax = axis_nb(x, a.nx, -1, -1), ay = axis_nb(y, a.ny, -1, -1), az = axis_nb(z, a.nz, -1, -1);
    R mx = R(0), my = R(0), mz = R(0);
    unsigned src[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) {
      src[i] = un + (unsigned)((ax.idx[2 - cx(i)] - x) + (ay.idx[2 - cy(i)] - y) * a.nx + (az.idx[2 - cz(i)] - z) * nxy);
      const R gi = decode<R>(ldg(pin + (size_t)i * N, src[i]));
      if (cx(i)) mx += R(cx(i)) * gi;
      if (cy(i)) my += R(cy(i)) * gi;
      if (cz(i)) mz += R(cz(i)) * gi;
    }
    const R rho0 = a.th.rho_ref;
    const R mom = fdiv(a.P0, s * rho0);
    const R ux = mx * mom, uy = my * mom, uz = mz * mom;
    const R T = NS ? (R)((const Sc *)a.scal_in)[n] : R(0);
    if (pass == 0) {
      red[0] = 0.5 * (double)rho0 * ((double)ux * ux + (double)uy * uy + (double)uz * uz);
      red[1] = (double)T;
      red[2] = (double)T * (double)T;
    } else {
      // dJ/dA_i at the pull source of link i: rho mom (c_i . u)
#pragma unroll
      for (int i = 0; i < 27; ++i)
        stg(lamA + (size_t)i * N, src[i], rho0 * mom * (R(cx(i)) * ux + R(cy(i)) * uy + R(cz(i)) * uz));
      if (NS) lamT[n] = R(2) * (T - R(mean_T));
    }
  }
  if (pass == 0) block_sums(red, a.partials + (size_t)blockIdx.x * NSUM);
}

// Reverse of the equilibrium initialisation (Eq. 6) with respect to u0 (FP64 fields).
template <int PREC>
__global__ __launch_bounds__(256) void init_adjoint_kernel(KArgs<double> a, const typename Prec<PREC>::R *lamA,
                                                           const double *u0, double *gu) {
  const int n = blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
  const int N = a.N;
  if (n >= N) return;
  const double ux = u0[n], uy = u0[N + n], uz = u0[2 * N + n];
  const double kq = a.th.rho_ref * (1.0 / 3.0) / a.P0;
  double gx = 0.0, gy = 0.0, gz = 0.0;
  for (int i = 0; i < 27; ++i) {
    const double l = (double)lamA[(size_t)i * N + n] * wgt<27>(i) * kq;
    const double cu = cx(i) * ux + cy(i) * uy + cz(i) * uz;
    gx += l * (3.0 * cx(i) + 9.0 * cu * cx(i) - 3.0 * ux);
    gy += l * (3.0 * cy(i) + 9.0 * cu * cy(i) - 3.0 * uy);
    gz += l * (3.0 * cz(i) + 9.0 * cu * cz(i) - 3.0 * uz);
  }
  gu[n] = gx;
  gu[N + n] = gy;
  gu[2 * N + n] = gz;
}

template <class T> __global__ void convert_kernel(const T *in, double *out, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (double)in[i];
}

template <int PREC>
hipError_t launch_adjoint_p(int ns, int kind, const StepArgs &sa, int nblocks, hipStream_t st, const void *p0,
                            const void *p1, void *p2, void *p3, void *p4, double mean_T, const double *u0, double *gu) {
  using R = typename Prec<PREC>::R;
  KArgs<R> a = to_kargs<R>(sa);
  if (kind == 0) {   // adjoint step
    // XCD order where there is more than about a block a CU: a few blocks gain nothing from shared
    // planes and pay for the order (us per step, linear / XCD order: FP64 24^3 12.0 / 12.5, 40^3 16.2 /
    // 15.7, 80^3 110 / 100)
    a.remap = nblocks > 192;
    // NT: FP32 steps whose arrays exceed the 256 MB Infinity Cache.  Those of a smaller grid stay
    // there from one reverse step to the next (us per step, kept / streamed: passive 64^3 25.7 /
    // 27.0, 96x64x96 (260 MB) 47.2 / 52.4, 96^3 (389 MB) 78.9 / 72.5, 128^3 191.7 / 187.9; isothermal
    // 96x64x96 33.8 / 37.6, 96^3 (287 MB) 57.1 / 52.3, 128^3 141.9 / 138.5; FP64 passive 128^3 435 / 447)
    const size_t bytes = (size_t)sa.N * sizeof(R) * (ns ? 110 : 81);
    const bool nt = PREC != 0 && bytes > ((size_t)256 << 20);
    auto run = [&](auto scalars, auto stream) {
      hipLaunchKernelGGL((adjoint_kernel<PREC, decltype(scalars)::value, PREC != 0 && decltype(stream)::value>),
                         dim3(nblocks), dim3(256), 0, st, a, (const R *)p0, (const R *)p1, (R *)p2, (R *)p4);
    };
    auto run_ns = [&](auto scalars) { nt ? run(scalars, std::true_type{}) : run(scalars, std::false_type{}); };
    if (ns == 0) {
      run_ns(std::integral_constant<int, 0>{});
    } else {
      run_ns(std::integral_constant<int, 1>{});
      hipLaunchKernelGGL((adjoint_scalar_kernel<PREC>), dim3(nblocks), dim3(256), 0, st, a, (const R *)p1, (const R *)p4,
                         (R *)p3);
    }
  } else if (kind == 1 || kind == 2) {   // objective pass 0 (sums) / pass 1 (gradient)
    if (ns == 0)
      hipLaunchKernelGGL((objective_kernel<PREC, 0>), dim3(nblocks), dim3(256), 0, st, a, mean_T, kind - 1, (R *)p2,
                         (R *)p3);
    else
      hipLaunchKernelGGL((objective_kernel<PREC, 1>), dim3(nblocks), dim3(256), 0, st, a, mean_T, kind - 1, (R *)p2,
                         (R *)p3);
  } else {   // init adjoint
    hipLaunchKernelGGL((init_adjoint_kernel<PREC>), dim3(nblocks), dim3(256), 0, st, to_kargs<double>(sa),
                       (const R *)p0, u0, gu);
    if (ns && p3)
      hipLaunchKernelGGL((convert_kernel<R>), dim3((sa.N + 255) / 256), dim3(256), 0, st, (const R *)p1, (double *)p3,
                         (long long)sa.N);
  }
  return hipGetLastError();
}

hipError_t launch_adjoint(int prec, int ns, int kind, const StepArgs &sa, int nblocks, hipStream_t st, const void *p0,
                          const void *p1, void *p2, void *p3, void *p4, double mean_T, const double *u0,
                          double *gu) {
  if (prec == 0) return launch_adjoint_p<0>(ns, kind, sa, nblocks, st, p0, p1, p2, p3, p4, mean_T, u0, gu);
  return launch_adjoint_p<1>(ns, kind, sa, nblocks, st, p0, p1, p2, p3, p4, mean_T, u0, gu);
}

}  // namespace lbm
