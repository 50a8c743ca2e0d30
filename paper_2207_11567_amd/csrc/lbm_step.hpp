// Fused time-step kernel of the hybrid LB/FD scheme (one thread per cell) and the
// auxiliary kernels (geometry words, equilibrium initialisation, FP64 sum finalisation).
//
// Per fluid cell, in one pass:
//   scalars at the cell and its axis neighbours (ghost rules at walls, inlet, outlet)
//   -> rho (ideal gas), grad rho, diffusion + reaction right-hand sides, Lambda (Eq. 3)
//   -> pull-streaming of the Q populations with boundary substitutions (Eq. 1)
//   -> moments P_h, u (Eq. 7) -> WENO3 advection, explicit Euler scalar update (Sec. 2.3)
//   -> source Xi (Eq. 2) -> pre-conditioning (Eq. 13) -> cumulant collision (Eqs. 9-12,
//      optionally with Geier's Galilean correction)
//   -> post-collision populations (Eq. 8) stored as deviations from the lattice weights
//   -> FP64 block partial sums (wavefront shuffles + LDS), one record per block.
// In a closed domain the thermodynamic pressure P_th = pi P_th(0) scales the ideal-gas
// density, its rate q = dln(pi)/dt adds the pressure work kappa T q to the temperature
// right-hand side and shifts Lambda to the velocity divergence Lambda - q, and the
// finalisation of the sums sets pi for the next step from the mass the domain holds.
// With a signed wall distance bound (curved walls), links from solid cells use the
// linearly interpolated bounce-back and scalar stencil points in solid cells take the
// value at their mirror image about the wall (boundary cells only).
#pragma once

#include <type_traits>

#include "lbm_device.hpp"

namespace lbm {

// Per-block FP64 sums: rho, P_h, rho u (3), rho |u|^2/2, W/T, rho Y_1 at level n, and
// W/T of the updated scalars (level n+1; formed in closed domains only).
constexpr int NSUM = 9;
// collision operator compiled into a step instance
enum : int { COLL_CUM1 = 0, COLL_CUM = 1, COLL_BGK = 2 };
// cells that step_cells updates: every cell (64x4 tile grid when it fits, else linear
// 256-cell tiles), the interior cells only (the code of boundaries, solids and curved walls
// is not compiled in; on the tile grid, where a wave's y and z are scalars, or on linear
// tiles for grids the tiles do not fit), or the cells of a list (one thread per listed
// cell: the cells the interior code leaves); or every cell of a domain without boundaries
// (all faces periodic, no solids: nothing but interior cells, on the tile grid or on linear
// tiles)
enum : int { MODE_ALL = 0, MODE_INTERIOR = 1, MODE_LIST = 2, MODE_INTERIOR_LIN = 3, MODE_FREE = 4, MODE_FREE_LIN = 5 };

// Host-side description of one launch (double precision constants).
struct Thermo {
  double rho_ref, T_ref, nu_ref, inv_Pr, F, visc_const_mu;
  double chem[32];
};

struct StepArgs {
  const void *pop_in;
  void *pop_out;
  const void *scal_in;
  void *scal_out;
  const void *geom;    // per-cell geometry words or nullptr
  double *partials;    // [nblocks][NSUM]
  int *flag;           // bit 0: non-finite value seen
  const double *thermo;  // closed domain: device (pi, q, K); nullptr when P_th is constant
  double kappa;        // (gamma - 1)/gamma
  const double *lvl;   // signed wall distance per node (curved walls) or nullptr
  double *stats;       // running statistics [2(D+1)][N] (means, then sums of squared
                       // deviations) of u_d and P_h - P0, or nullptr when not sampled
  double inv_k;        // 1/k for the k-th sample
  double *probe_out;   // row of this level in the probe record ([nprobe][D+1]) or nullptr
  int nprobe;
  int probe[8];        // probe cells
  int mix;             // mixture-averaged transport (two-step scalars)
  double transport[32];  // binary D0 (15), c_p a_k (6), b_k (6), exponents of mu and D
  double mix_in[19];   // inlet transport point: lambda, rho D_k W_k/W (6), X_k (6), Y_k (6)
  double *f_P, *f_rho, *f_u, *f_scal;   // field outputs (extract mode)
  const int *cells;    // split step: linear indices of the boundary cells
  int ncells;
  int nlb;             // blocks that update them (a multiple of 8)
  int nx, ny, nz;
  long long N;
  int face[6];         // ST_* code of each face, -1 for periodic
  long long step;
  int collision;       // 0 cumulant, 1 BGK
  int gal;             // Galilean correction of the cumulant collision
  int p4;              // D3Q27 parameterised higher-order relaxation (fourth-order diffusion)
  int remap;           // XCD-aware block order
  int band_rows;       // 0: linear 256-cell tiles; else 64x4 tiles in bands of this many rows
  int pull_cached;     // production instance with cached pull loads (else streaming loads)
  double P0;           // rho_ref cs2
  double wb, wh, smag18;
  double inlet_u[3], inlet_noise, outlet_P;
  double phi_in[8];    // inlet scalars
  double eps[8];       // WENO eps per scalar
  unsigned long long seed;
  Thermo th;
};

// Kernel arguments with every floating constant already in the compute precision R, so
// that the kernel reads uniform values straight from the argument segment.
template <class R> struct KArgs {
  const void *pop_in;
  void *pop_out;
  const void *scal_in;
  void *scal_out;
  const void *geom;
  double *partials;
  int *flag;
  const double *thermo;
  const double *lvl;
  double *stats;
  double inv_k;
  double *probe_out;
  int nprobe;
  int probe[8];
  double *f_P, *f_rho, *f_u, *f_scal;
  const int *cells;
  int ncells, nlb;     // split step: listed boundary cells and the blocks that update them
  int nx, ny, nz, N;
  int face[6];
  long long step;
  int collision, remap, band_rows, gal, p4;
  int big;             // a population copy exceeds the 256 MB Infinity Cache
  R P0, invP0, wb, wh, smag18, kap;
  R inlet_u[3], outlet_P;
  double inlet_noise;
  R phi_in[8], eps[8];
  unsigned long long seed;
  double inv_T_ref_d, W_d[6];
  double P0d;          // P0 in FP64 (field outputs and sums of P_h)
  ThermoT<R> th;
  MixT<R> mx;
};

// The step kernels read their arguments where the launch put them (constant memory, scalar
// loads at each use): a parameter handed on by reference is first copied field by field, all
// of it loaded up front into scalar registers that the long kernels then spill.
template <class R> __device__ __forceinline__ const KArgs<R> &kernel_args() {
  return *(const KArgs<R> *)__builtin_amdgcn_kernarg_segment_ptr();
}

template <class R> KArgs<R> to_kargs(const StepArgs &a) {
  KArgs<R> k;
  k.pop_in = a.pop_in; k.pop_out = a.pop_out; k.scal_in = a.scal_in; k.scal_out = a.scal_out;
  k.geom = a.geom; k.partials = a.partials; k.flag = a.flag; k.thermo = a.thermo; k.lvl = a.lvl;
  k.stats = a.stats; k.inv_k = a.inv_k; k.probe_out = a.probe_out; k.nprobe = a.nprobe;
  for (int j = 0; j < 8; ++j) k.probe[j] = a.probe[j];
  k.kap = (R)a.kappa;
  k.f_P = a.f_P; k.f_rho = a.f_rho; k.f_u = a.f_u; k.f_scal = a.f_scal;
  k.cells = a.cells; k.ncells = a.ncells; k.nlb = a.nlb;
  k.nx = a.nx; k.ny = a.ny; k.nz = a.nz; k.N = (int)a.N;
  for (int f = 0; f < 6; ++f) k.face[f] = a.face[f];
  k.step = a.step; k.collision = a.collision; k.remap = a.remap; k.band_rows = a.band_rows;
  k.big = a.pull_cached;
  k.gal = a.gal;
  k.p4 = a.p4;
  k.P0 = (R)a.P0; k.invP0 = (R)(1.0 / a.P0); k.wb = (R)a.wb; k.wh = (R)a.wh; k.smag18 = (R)a.smag18;
  for (int d = 0; d < 3; ++d) k.inlet_u[d] = (R)a.inlet_u[d];
  k.outlet_P = (R)a.outlet_P; k.inlet_noise = a.inlet_noise;
  for (int q = 0; q < 8; ++q) { k.phi_in[q] = (R)a.phi_in[q]; k.eps[q] = (R)a.eps[q]; }
  k.seed = a.seed;
  const double *ch = a.th.chem;
  k.inv_T_ref_d = 1.0 / a.th.T_ref;
  k.P0d = a.P0;
  for (int q = 0; q < 6; ++q) k.W_d[q] = ch[5 + q] > 0.0 ? ch[5 + q] : 1.0;
  ThermoT<R> &t = k.th;
  t.rho_ref = (R)a.th.rho_ref; t.nu_ref = (R)a.th.nu_ref; t.mu_ref = (R)(a.th.nu_ref * a.th.rho_ref);
  t.inv_Pr = (R)a.th.inv_Pr; t.F = (R)a.th.F; t.invF = (R)(1.0 / a.th.F);
  t.const_mu = a.th.visc_const_mu != 0.0;
  t.rhoT = (R)(a.th.rho_ref * a.th.T_ref);
  t.rhoT_W = (R)(ch[17] > 0.0 ? a.th.rho_ref * a.th.T_ref / ch[17] : 0.0);
  t.B1 = (R)ch[0]; t.Ta1 = (R)ch[1]; t.B2 = (R)ch[2]; t.Ta2 = (R)ch[3];
  t.heat1 = (R)(ch[4] > 0.0 ? (ch[3] - ch[2]) / ch[4] : 0.0);
  t.inv_cp = (R)(ch[4] > 0.0 ? 1.0 / ch[4] : 0.0);
  for (int q = 0; q < 6; ++q) {
    t.W[q] = (R)ch[5 + q];
    t.inv_W[q] = (R)(ch[5 + q] > 0.0 ? 1.0 / ch[5 + q] : 0.0);
    t.h[q] = (R)ch[11 + q];
  }
  for (int q = 0; q < 5; ++q)
    t.dinv_W[q] = (R)(ch[5 + q] > 0.0 && ch[10] > 0.0 ? 1.0 / ch[5 + q] - 1.0 / ch[10] : 0.0);
  MixT<R> &m = k.mx;
  m.on = a.mix;
  const double *tr = a.transport;
  for (int i = 0, n = 0; i < 6; ++i) {
    m.invB[i][i] = R(0);
    for (int j = i + 1; j < 6; ++j, ++n) m.invB[i][j] = m.invB[j][i] = (R)(tr[n] > 0.0 ? 1.0 / tr[n] : 0.0);
  }
  const double T0 = 298.15;     // reference temperature of the formation enthalpies
  for (int q = 0; q < 6; ++q) {
    m.cpa[q] = (R)tr[15 + q];
    m.cpb[q] = (R)tr[21 + q];
    m.hc[q] = (R)(ch[11 + q] - ch[5 + q] * (tr[15 + q] * T0 + 0.5 * tr[21 + q] * T0 * T0));
  }
  m.s_mu = (R)tr[27];
  m.s_D = (R)tr[28];
  m.inv_Tref = (R)(1.0 / a.th.T_ref);
  m.in_kap = (R)a.mix_in[0];
  for (int q = 0; q < 6; ++q) {
    m.in_coef[q] = (R)a.mix_in[1 + q];
    m.in_X[q] = (R)a.mix_in[7 + q];
    m.in_Y[q] = (R)a.mix_in[13 + q];
  }
  return k;
}

template <int Q> struct GeomWord { using T = uint64_t; };
template <> struct GeomWord<9> { using T = uint32_t; };
// bit i < Q: the source cell of link i is solid; bit Q: the cell itself is solid;
// bit Q+1+2d (+1): the cell at +2 e_d (-2 e_d) is solid.
template <int Q> __host__ __device__ constexpr int bit_self() { return Q; }
template <int Q> __host__ __device__ constexpr int bit_far(int d, int neg) { return Q + 1 + 2 * d + neg; }

// Links (one bit each) whose source lies one cell further along axis d, at -1 (side 0) or +1.
template <int Q> __host__ __device__ constexpr unsigned links_from(int d, int side) {
  unsigned m = 0;
  for (int i = 0; i < Q; ++i) {
    const int c = d == 0 ? cx(i) : d == 1 ? cy(i) : Q == 27 ? cz(i) : 0;
    if (c == (side == 0 ? 1 : -1)) m |= 1u << i;
  }
  return m;
}

// XCD-aware block order: hardware hands consecutive workgroups to the 8 XCDs in turn;
// remapping gives each XCD a contiguous slab of cells so that halo rows shared between
// neighbouring blocks stay in the same L2.
__device__ __forceinline__ int tile_of_block(int b, int nb, int remap) {
  if (!remap) return b;
  const int per = nb / 8;
  if (b >= per * 8) return b;
  return (b % 8) * per + b / 8;
}

__device__ __forceinline__ double splitmix_xi(unsigned long long seed, unsigned long long a,
                                              unsigned long long b, unsigned long long n) {
  unsigned long long z = seed + ((n << 40) | (b << 20) | a) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const double U = (double)(z >> 11) * 0x1.0p-53;
  return 1.7320508075688772 * (2.0 * U - 1.0);
}

// Per-axis neighbour coordinates k = -2..2 with periodic wrap; out-of-domain positions
// through a non-periodic face get the face's status code.
struct AxisNb {
  int idx[5];
  int code[5];   // -1: inside (or wrapped), else ST_SOLID / ST_INLET / ST_OUTLET
};
__device__ __forceinline__ AxisNb axis_nb(int c, int n, int flo, int fhi) {
  AxisNb r;
#pragma unroll
  for (int k = -2; k <= 2; ++k) {
    int p = c + k;
    int code = -1;
    if (p < 0) {
      if (flo < 0) p += n; else code = flo;
    } else if (p >= n) {
      if (fhi < 0) p -= n; else code = fhi;
    }
    // extents of one cell: wrap a second time (|k| <= 2), no division
    if (code < 0) {
      if (p < 0) p += n;
      if (p >= n) p -= n;
    }
    r.idx[k + 2] = code < 0 ? p : c;
    r.code[k + 2] = code;
  }
  return r;
}

// Offsets (times the axis stride) and face codes of positions c-2..c+2 on one axis; cells at
// least two away from both ends take the plain offsets without any wrap logic.
__device__ __forceinline__ void axis_offsets(int c, int n, int flo, int fhi, int stride, int (&off)[5],
                                             int (&code)[5]) {
  if (c >= 2 && c < n - 2) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      off[k] = (k - 2) * stride;
      code[k] = -1;
    }
  } else if (flo < 0 && fhi < 0) {
    // periodic axis: the wrap alone, by selects (twice, for extents of one cell)
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      int p = c + k - 2;
      p += p < 0 ? n : 0;
      p -= p >= n ? n : 0;
      p += p < 0 ? n : 0;
      p -= p >= n ? n : 0;
      off[k] = (p - c) * stride;
      code[k] = -1;
    }
  } else {
    const AxisNb A = axis_nb(c, n, flo, fhi);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      off[k] = (A.idx[k] - c) * stride;
      code[k] = A.code[k];
    }
  }
}

// A cell needs the general (boundary) code when its geometry word is not zero (it is
// solid, or a solid lies within its links or its +-2 stencil) or a non-periodic face lies
// within two cells on some axis; every other cell is interior.  The host builds the list
// of general cells with the same rule (lbm_capi.hip), so the interior and list instances
// of a step cover every cell exactly once.
__device__ __forceinline__ bool near_face(int c, int n, int flo, int fhi) {
  return (flo >= 0 && c < 2) || (fhi >= 0 && c >= n - 2);
}

// Element access through a wave-uniform base pointer and a 32-bit byte offset, so that
// the compiler can address with the scalar base + vector offset form.
template <class T> __device__ __forceinline__ T ldg(const T *base, unsigned idx) {
  return *(const T *)((const char *)base + idx * (unsigned)sizeof(T));
}
template <class T> __device__ __forceinline__ void stg(T *base, unsigned idx, T v) {
  *(T *)((char *)base + idx * (unsigned)sizeof(T)) = v;
}

// Element of an array of up to 2^31 elements (64-bit byte address).
template <class T> __device__ __forceinline__ T ldg64(const T *base, unsigned idx) { return base[(size_t)idx]; }

// Raw buffer access: one descriptor (SGPRs) per array slice (a population or a scalar
// field, under 4 GiB since Q N < 2^31 elements) and a 32-bit byte offset per lane, so the
// neighbours of a cell share offset registers and no load needs 64-bit address arithmetic.
// AUX 2 marks a streaming (non-temporal) access.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slice(const void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, -1, 0x00020000);
}
template <class T, int AUX = 0> __device__ __forceinline__ T bld(__amdgpu_buffer_rsrc_t r, unsigned idx) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, idx * 8u, 0, AUX));
  else if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, idx * 4u, 0, AUX));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, idx * 2u, 0, AUX));
}
template <class T, int AUX = 0> __device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, unsigned idx, T v) {
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, idx * 8u, 0, AUX);
  else if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, idx * 4u, 0, AUX);
  else
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, idx * 2u, 0, AUX);
}

// (1 - p) a + p b, exact at p = 0 and p = 1.
template <class R> __device__ __forceinline__ R lerp(R a, R b, R p) { return (R(1) - p) * a + p * b; }

// Interpolation weight toward the second node for a mirror image at distance p <= 1 from
// the first fluid node: p itself, or, for an image between the wall and that node
// (p < 0), the even quadratic through the two nodes (zero gradient at the wall).
template <class R> __device__ __forceinline__ R image_weight(R p) { return p >= R(0) ? p : fdiv(p, R(2) - p); }


// Block reduction of NSUM doubles into partials[tile*NSUM ..] in a fixed order: every
// thread parks its values in LDS, then thread t < 8 NSUM sums 32 cells of counter t/8, and
// the 8 threads of each counter (aligned groups inside one wave) combine by xor-shuffles.
// 256 threads per block.
__device__ __forceinline__ void block_sums(double (&v)[NSUM], double *out) {
  __shared__ double sh[NSUM][256];
  const int t = threadIdx.x;
  const int slot = (t & 31) * 8 + (t >> 5);          // part (t>>5) of 8, element t&31
#pragma unroll
  for (int k = 0; k < NSUM; ++k) sh[k][slot] = v[k];
  __syncthreads();
  if (t < 8 * NSUM) {
    const int k = t >> 3, part = t & 7;
    double acc = 0.0;
#pragma unroll 8
    for (int j = 0; j < 32; ++j) acc += sh[k][j * 8 + part];
    acc += __shfl_xor(acc, 4, 64);
    acc += __shfl_xor(acc, 2, 64);
    acc += __shfl_xor(acc, 1, 64);
    if (part == 0) out[k] = acc;
  }
}

// W/T of a cell up to a constant factor (the density per unit thermodynamic pressure):
// 1/T_ref without a temperature, 1/T for the one-step model's constant W.
template <int NS, class R>
__device__ __forceinline__ double w_over_T(const ThermoT<R> &t, const R (&v)[NS > 0 ? NS : 1], double inv_T_ref) {
  if constexpr (NS <= 1) {
    return inv_T_ref;
  } else if constexpr (NS == 2) {
    return (double)fdiv(R(1), v[0]);
  } else {
    R inv = t.inv_W[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) inv += v[1 + q] * t.dinv_W[q];
    return (double)fdiv(R(1), inv * v[0]);
  }
}

// FULL: the instance that also carries curved walls (a.lvl) and the observables
// (a.stats, a.probe_out), each switched on by its pointer; the plain instances carry none
// of that code, so their register allocation is that of the bare step.
// COLL: the collision compiled in: COLL_CUM1 cumulant with every order >= 3 relaxed at
// rate one (D3Q27; any rate on D2Q9), COLL_CUM general cumulant rates, COLL_BGK the BGK
// test mode.  Each instance holds one operator, so the registers of the unused ones do not
// count against the production path.
// The cells of one block of a step: red gets each thread's contribution to the FP64 sums,
// the return value is the block's place among its kind (tile, or list block).
template <int Q, int PREC, int NS, bool EXTRACT, bool FULL, int COLL, int MODE, bool PULLC>
__device__ __forceinline__ int step_cells(const KArgs<typename Prec<PREC>::R> &a, int block, int nblocks,
                                          double (&red)[NSUM]) {
#include "lbm_step_cells.inc"
  return tile;
}

// One kind of cell per launch: every cell, or one half of a split step of D3Q27 (interior
// tiles, or the listed boundary cells, two kernels side by side on two streams).
// The FP32-arithmetic two-step D3Q27 step (FP32 or FP16 storage) asks for four waves per
// SIMD (at most 128 VGPRs): its allocation otherwise lands a few registers above that, at
// three waves; the few spilled values cost less than the lost wave (measured 9 % faster on
// the reacting box in both storage precisions, 12 % for the interior half of the step
// with mixture-averaged transport).  Its list half asks for the same, so that one of its
// waves fits the place that an interior wave leaves.  The all-cell D3Q27 instances ask for the
// waves that their interior cells can use: the scheduler otherwise spends registers on the
// loads in flight that only the boundary cells issue.
template <int Q, int PREC, int NS, bool EXTRACT, bool FULL, int COLL, int MODE>
constexpr int step_waves_per_eu() {
  if (Q != 27 || EXTRACT || COLL != COLL_CUM1) return 1;
  if (MODE == MODE_LIST) return PREC != 0 && NS == 6 ? (FULL ? 3 : 4) : 1;
  if (MODE == MODE_ALL) {
    if (PREC == 0) return NS == 0 ? (FULL ? 4 : 5) : NS == 1 ? (FULL ? 3 : 4) : NS == 2 ? 2 : 1;
    return NS == 0 ? (FULL ? 6 : 8) : NS == 1 ? (FULL ? 5 : 6) : NS == 2 ? (FULL ? 4 : 5) : (FULL ? 3 : 4);
  }
  return PREC != 0 && NS == 6 ? 4 : 1;
}
// SEG: the arguments are read where the launch put them, through step_cells, instead of as the
// kernel's parameter; the same formulas, another register allocation (118 instead of 112
// VGPRs, other places of the loads).  Measured per kind of step: faster for the interior cells of
// the two-step step (reacting box 192x192x384 FP32 843 -> 827 us, FP16 storage 713 -> 681) and
// for HIT 256^3 with FP16 storage (378 -> 365), slower beside the curved-wall list (cone
// 128x128x256 298 -> 330: its waves no longer fit beside three interior ones).
template <int Q, int PREC, int NS, bool EXTRACT, bool FULL, int COLL, int MODE, bool PULLC = false, bool SEG = false>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(step_waves_per_eu<Q, PREC, NS, EXTRACT, FULL, COLL, MODE>())))
void step_kernel(KArgs<typename Prec<PREC>::R> a) {
  double red[NSUM] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  if constexpr (SEG) {
    const auto &ka = kernel_args<typename Prec<PREC>::R>();
    const int tile = step_cells<Q, PREC, NS, EXTRACT, FULL, COLL, MODE, PULLC>(ka, blockIdx.x, gridDim.x, red);
    block_sums(red, ka.partials + (size_t)tile * NSUM);
  } else {
    const int block = (int)blockIdx.x, nblocks = (int)gridDim.x;
#include "lbm_step_cells.inc"
    block_sums(red, a.partials + (size_t)tile * NSUM);
  }
}

// D2Q9: a step split by kind of cell in one launch.  The first a.nlb blocks (a multiple of
// 8, so that the tiles' blocks keep their XCDs) update the listed boundary cells, the others
// the interior cells of their tile.  Both kinds need the same registers here, so one
// kernel costs no occupancy, the long boundary chains start first and end under the interior
// ones, and nothing waits for another stream's event.  With observables or mixture transport in
// the two-step step the two bodies together took a wave more than one does (FP64 one wave per
// SIMD instead of two, FP32 three instead of four), so these ask for it: channel 2048x512 with
// mixture transport FP64 225 -> 145 us per step (163 as one instance), FP32 70 -> 63 (75).
template <int PREC, int NS, bool LFULL, bool IFULL, int COLL, int IMODE, bool PULLC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(IFULL && NS == 6 ? (PREC == 0 ? 2 : 4) : 1)))
void split_kernel(KArgs<typename Prec<PREC>::R>) {
  const auto &a = kernel_args<typename Prec<PREC>::R>();
  double red[NSUM] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const int block = (int)blockIdx.x - a.nlb, ntiles = (int)gridDim.x - a.nlb;
  int rec;
  if (block < 0) {
    rec = ntiles + step_cells<9, PREC, NS, false, LFULL, COLL, MODE_LIST, false>(a, blockIdx.x, a.nlb, red);
  } else {
    rec = step_cells<9, PREC, NS, false, IFULL, COLL, IMODE, PULLC>(a, block, ntiles, red);
  }
  block_sums(red, a.partials + (size_t)rec * NSUM);
}

// The first bytes of the work buffer (divergence flag at 0, final sums at 64, thermodynamic
// pressure at 192): 32 doubles that the synchronising calls hand to the host, written by a
// kernel of the call straight into the solver's pinned host copy, where it has one (a
// device-to-host copy of each piece cost a launch and a staging wait of its own).
constexpr int HEAD_WORDS = 32, HEAD_SUMS = 8;

// Deterministic reduction of block records, nrec x W doubles (W = NSUM counters, or one) read
// as one contiguous run: thread t of the first 1017 (the largest multiple of NSUM; all 1024
// for one counter) adds elements t, t + 1017, ..., all of one counter, then wave k combines
// counter k.  Each block sums `chunk` records; the order of
// every addition is fixed by the launch shape, so results are bitwise repeatable.  With a
// host copy (one block, out in the work buffer's head) the whole head goes there too.
// Records read as rows of NSUM by 256 threads and summed in two launches took 9 us for the
// 1024..4900 records of the 2-D workloads, this one 4 to 6.
template <int W>
static __global__ __launch_bounds__(1024) void reduce_records(const double *in, int nrec, int chunk, double *out,
                                                              const double *head, double *host) {
  constexpr int USED = 1024 / W * W, GROUPS = USED / W;
  __shared__ double sh[USED];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const long long b0 = (long long)blockIdx.x * chunk;
  const int count = (int)min((long long)chunk, nrec - b0) * W;
  const double *rec = in + b0 * W;
  if (t < USED) {
    double acc = 0.0;
#pragma unroll 8
    for (int e = t; e < count; e += USED) acc += rec[e];
    sh[t] = acc;
  }
  __syncthreads();
  if (w < W) {
    double acc = 0.0;
    for (int j = lane; j < GROUPS; j += 64) acc += sh[j * W + w];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) {
      out[(size_t)blockIdx.x * W + w] = acc;
      if (host) host[HEAD_SUMS + w] = acc;
    }
  }
  if (host && t < HEAD_WORDS && (t < HEAD_SUMS || t >= HEAD_SUMS + W)) host[t] = head[t];
}

// The head alone, for calls without a kernel that could pass it on.
static __global__ void publish_kernel(const double *head, double *host) {
  if (threadIdx.x < HEAD_WORDS) host[threadIdx.x] = head[threadIdx.x];
}

// State copy: two arrays of 16-byte words in one launch, four words in flight per thread, and
// the head for the host.  Streaming where the copy exceeds the Infinity Cache (get_state of
// the 192x192x384 FP32 reacting box 0.78 ms as the runtime's copies, 4.7 TB/s).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ __forceinline__ void copy_words(const u32x4 *src, u32x4 *dst, size_t n, size_t i, size_t stride) {
  for (; i + 3 * stride < n; i += 4 * stride) {
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = STREAM ? __builtin_nontemporal_load(src + i + j * stride) : src[i + j * stride];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (STREAM) __builtin_nontemporal_store(v[j], dst + i + j * stride);
      else dst[i + j * stride] = v[j];
  }
  for (; i < n; i += stride) dst[i] = src[i];
}
template <bool STREAM>
__global__ __launch_bounds__(256) void copy_state_kernel(const u32x4 *a, u32x4 *da, size_t na, const u32x4 *b, u32x4 *db,
                                                         size_t nb, const double *head, double *host) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
  if (host && i < HEAD_WORDS) host[i] = head[i];
  copy_words<STREAM>(a, da, na, i, stride);
  copy_words<STREAM>(b, db, nb, i, stride);
}

// Closed domain, after every step: (pi, q, K) advanced from the two sums it needs, sum W/T
// at level n and of the updated scalars (record entries 6 and 8), in one block of 1024
// threads: thread t adds records t, t + 1024, ..., then the lanes of each wave by a
// butterfly (lane 0's value kept) and the 16 waves in order.  A fixed order of additions,
// so the result is bitwise repeatable; one short kernel over two of the NSUM entries.
static __global__ __launch_bounds__(1024) void thermo_kernel(const double *rec, int nrec, double *thermo) {
  __shared__ double part[2][16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  double s6 = 0.0, s8 = 0.0;
  for (int b = t; b < nrec; b += 1024) {
    s6 += rec[(size_t)b * NSUM + 6];
    s8 += rec[(size_t)b * NSUM + 8];
  }
  for (int o = 32; o > 0; o >>= 1) {
    s6 += __shfl_xor(s6, o, 64);
    s8 += __shfl_xor(s8, o, 64);
  }
  if (lane == 0) {
    part[0][w] = s6;
    part[1][w] = s8;
  }
  __syncthreads();
  if (t == 0) {
    double a6 = 0.0, a8 = 0.0;
    for (int j = 0; j < 16; ++j) {
      a6 += part[0][j];
      a8 += part[1][j];
    }
    const double pi = thermo[0];
    double K = thermo[2];
    if (!(K > 0.0)) K = pi * a6;
    const double pn = K / a8;
    thermo[0] = pn;
    thermo[1] = (pn - pi) / pi;
    thermo[2] = K;
  }
}

// (pi, q, K) set from the host's values (a kernel rather than a copy, so that the call
// needs no host buffer to outlive it).
static __global__ void set_thermo_kernel(double *thermo, double pi, double q, double K) {
  if (threadIdx.x == 0) {
    thermo[0] = pi;
    thermo[1] = q;
    thermo[2] = K;
  }
}

// Generalised flame surface: |grad c| summed over fluid cells, c = (T - T_u)/(T_b - T_u),
// central differences with the ghost rules of grad rho (own value across walls, solids
// and the outlet, the inlet temperature across the inlet); one FP64 record per block.  The
// neighbours are loads from selected addresses, and the block sums one value by shuffles
// instead of NSUM of them through LDS.
template <int Q, int PREC>
__global__ __launch_bounds__(256) void surface_kernel(KArgs<double> a, double inv_dT) {
  using Sc = typename Prec<PREC>::Sc;
  using GW = typename GeomWord<Q>::T;
  constexpr int D = Lat<Q>::D;
  __shared__ double part[4];
  const int n = tile_of_block(blockIdx.x, gridDim.x, a.remap) * 256 + (int)threadIdx.x;
  double acc = 0.0;
  if (n < a.N) {
    const GW gw = a.geom ? ((const GW *)a.geom)[n] : GW(0);
    const auto sT = slice(a.scal_in);
    const unsigned un = (unsigned)n;
    const int nxy = a.nx * a.ny, z = n / nxy, rem = n - z * nxy, y = rem / a.nx, x = rem - y * a.nx;
    double g2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      int off[5], code[5];
      axis_offsets(d == 0 ? x : d == 1 ? y : z, d == 0 ? a.nx : d == 1 ? a.ny : a.nz, a.face[2 * d], a.face[2 * d + 1],
                   d == 0 ? 1 : d == 1 ? a.nx : nxy, off, code);
      double v[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = s == 0 ? 3 : 1;                      // +1, -1
        const int bit = s == 0 ? link_from_plus<Q>(d) : link_from_minus<Q>(d);
        const bool own = code[k] >= 0 || ((gw >> bit) & 1);
        v[s] = (double)bld<Sc>(sT, own ? un : un + (unsigned)off[k]);
        if (code[k] == ST_INLET) v[s] = a.phi_in[0];
      }
      const double gd = 0.5 * (v[0] - v[1]) * inv_dT;
      g2 += gd * gd;
    }
    acc = gw & (GW(1) << bit_self<Q>()) ? 0.0 : sqrt(g2);
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) a.partials[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

// Mean and RMS fields from the running statistics (k samples): mean [D+1][N] (u_d, then
// P_h with P0 added back), rms = sqrt(M2/k).
static __global__ __launch_bounds__(256) void statistics_kernel(const double *acc, int D, long long N, double k,
                                                                 double P0, double *mean, double *rms) {
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  for (int j = 0; j <= D; ++j) {
    if (mean) mean[j * N + n] = acc[j * N + n] + (j == D ? P0 : 0.0);
    if (rms) rms[j * N + n] = sqrt(fmax(acc[(D + 1 + j) * N + n], 0.0) / k);
  }
}

__device__ __forceinline__ bool solid_at(const uint8_t *s, long long m) { return s[m] != 0; }
__device__ __forceinline__ bool solid_at(const double *phi, long long m) { return phi[m] < 0.0; }

// Geometry words from a solid mask, or from a signed wall distance (solid where < 0).
template <int Q, class Src>
__global__ __launch_bounds__(256) void geometry_kernel(const Src *solid, void *geom, int nx, int ny,
                                                        int nz, long long N, int f0, int f1, int f2,
                                                        int f3, int f4, int f5) {
  using GW = typename GeomWord<Q>::T;
  constexpr int D = Lat<Q>::D;
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int x = (int)(n % nx), y = (int)((n / nx) % ny), z = (int)(n / ((long long)nx * ny));
  const AxisNb ax = axis_nb(x, nx, f0, f1), ay = axis_nb(y, ny, f2, f3);
  const AxisNb az = D == 3 ? axis_nb(z, nz, f4, f5) : AxisNb{{z, z, z, z, z}, {-1, -1, -1, -1, -1}};
  auto lin = [&](int X, int Y, int Z) -> long long {
    return (long long)X + (long long)nx * ((long long)Y + (long long)ny * Z);
  };
  GW w = 0;
  if (solid_at(solid, n)) w |= GW(1) << bit_self<Q>();
  for (int i = 0; i < Q; ++i) {
    const int c[3] = {cx(i), cy(i), D == 3 ? cz(i) : 0};
    bool out = ax.code[2 - c[0]] >= 0 || ay.code[2 - c[1]] >= 0 || (D == 3 && az.code[2 - c[2]] >= 0);
    if (out || i == (Q - 1) / 2) continue;
    const long long m = lin(ax.idx[2 - c[0]], ay.idx[2 - c[1]], D == 3 ? az.idx[2 - c[2]] : z);
    if (solid_at(solid, m)) w |= GW(1) << i;
  }
  for (int d = 0; d < D; ++d) {
    const AxisNb &A = d == 0 ? ax : d == 1 ? ay : az;
    for (int neg = 0; neg < 2; ++neg) {
      const int k = neg ? 0 : 4;   // position -2 or +2
      if (A.code[k] >= 0) continue;
      const long long m = d == 0 ? lin(A.idx[k], y, z) : d == 1 ? lin(x, A.idx[k], z) : lin(x, y, A.idx[k]);
      if (solid_at(solid, m)) w |= GW(1) << bit_far<Q>(d, neg);
    }
  }
  ((GW *)geom)[n] = w;
}

// FP64 value to the storage precision, round to nearest even.  FP16 goes through FP32
// rounded to odd (the inexact bit kept in the last place), which the second rounding turns
// into the correct FP16: 8 instructions; the compiler's own conversion takes about 30.
template <class St> __device__ __forceinline__ St store_cast(double x) {
  if constexpr (sizeof(St) == 2) {
    const float f = (float)x;
    unsigned b = __builtin_bit_cast(unsigned, f);
    const double r = (double)f;
    if (r != x) b = (b - (fabs(r) > fabs(x) ? 1u : 0u)) | 1u;
    return (St)__builtin_bit_cast(float, b);
  } else {
    return (St)x;
  }
}

// Equilibrium initialisation (Eq. 6) from FP64 fields; populations stored as deviations.  The
// first thread also resets the thermodynamic pressure and the divergence flag.
template <int Q, int PREC, int NS>
__global__ __launch_bounds__(256) void init_kernel(KArgs<double> a, const double *Ph, const double *u,
                                                   const double *scal, double *thermo) {
  using P = Prec<PREC>;
  using St = typename P::St;
  using Sc = typename P::Sc;
  constexpr int D = Lat<Q>::D;
  constexpr int NSV = NS > 0 ? NS : 1;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    thermo[0] = 1.0;
    thermo[1] = thermo[2] = 0.0;
    *a.flag = 0;
  }
  const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long N = a.N;
  if (n >= N) return;
  double v[NSV];
  for (int k = 0; k < NSV; ++k) v[k] = 0.0;
  for (int k = 0; k < NS; ++k) {
    v[k] = scal[k * N + n];
    ((Sc *)a.scal_out)[k * N + n] = (Sc)v[k];
  }
  const double rho = density<NS, double>(a.th, v);
  const double ux = u[n], uy = u[N + n], uz = D == 3 ? u[2 * N + n] : 0.0;
  const double uu = ux * ux + uy * uy + uz * uz;
  const double ph1 = Ph[n] / a.P0 - 1.0;
  const double kq = rho * (1.0 / 3.0) / a.P0;
  for (int i = 0; i < Q; ++i) {
    const double cu = cx(i) * ux + cy(i) * uy + (D == 3 ? cz(i) * uz : 0.0);
    const double gh = wgt<Q>(i) * (ph1 + kq * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu));
    ((St *)a.pop_out)[i * N + n] = store_cast<St>(gh);
  }
}

}  // namespace lbm
