// gfx950 kernels of the 2D UGKS time step.
//
// One step is three launches on one stream (four in a periodic box):
//   ghost   periodic box only: the periodic images into the halo rows of every velocity plane
//   sums    per cell and velocity: limited slopes of f, the upwind reconstruction at the
//           cell's outgoing faces and their velocity moments (S1 and the sums of S7); in a
//           channel also the sums of the inlet and outlet ghost columns (Sec. 3.A)
//   faces   per interface: add the two sides' sums (and their parts, where a solver splits its
//           velocities into chunks), then the scalar part of the flux
//           (S2-S5: Maxwellian moments, time weights, micro slopes, equilibrium flux) into a
//           record of folded coefficients
//   update  per cell and velocity: the distribution flux at the faces (S6, S8), then Eq. (4)
//           for W and Eq. (3) for f; in a channel also the ghost states of the next step
//           (from W^{n+1}) and their Maxwellians in the ghost columns of f^{n+1}
// After the initial state and after a state is set, the update kernel's fill mode writes a
// channel's ghost columns from the current W.
// f is stored velocity-major: one plane per discrete velocity, a padded nx x ny array with
// two halo columns and rows on each side (KParams).  A wavefront takes 64 consecutive cells
// of one row at one velocity, so every load is one coalesced row segment and the x
// neighbours of a cell come from the neighbouring lanes.  The wavefronts of a workgroup share
// one row segment (the update kernel: the same segment of two rows) and take one velocity
// quadrant each (the FP64 update kernel: two wavefronts per quadrant, one per velocity
// chunk): within a quadrant the upwind direction of both axes is uniform, so an x-face flux
// is evaluated once, by the lane of its upwind cell, and handed to the downwind lane.
// Two variants run through the same kernels: a gas with internal degrees of freedom, whose
// second reduced distribution H takes velocity chunks of its own (its planes follow those of
// G), and the Shakhov collision model, a separate instantiation of the moment and update
// kernels (heat sums; equilibria times (1 + S)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <type_traits>

#include "ugks_internal.hpp"

namespace ugks {
namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kQuads = 4;                     // wavefronts per workgroup, one per quadrant
constexpr int kTileS = kWave - 2;             // cells per moment-kernel wavefront
constexpr int kTileU = kWave - 2 * kHalo;     // cells per update-kernel wavefront
constexpr unsigned kDropOffset = 0xFFFFFFF0u;  // beyond any plane (at most 2^31 bytes)

// Quadrant q of a workgroup: sign of u and of v.  Around the cycle (+,+) (-,+) (-,-) (+,-)
// neighbours share one sign, so each face side collects its sums from two adjacent waves.
__device__ __forceinline__ int quad_su(int q) { return (q == 0 || q == 3) ? 1 : -1; }
__device__ __forceinline__ int quad_sv(int q) { return q < 2 ? 1 : -1; }

// ------------------------------------------------------------------ storage
template <typename T>
__device__ __forceinline__ T ldb(const UGKS_GLOBAL T* p, unsigned byte_off) {
  return *reinterpret_cast<const UGKS_GLOBAL T*>(reinterpret_cast<const UGKS_GLOBAL char*>(p) +
                                                 byte_off);
}
template <typename S>
__device__ __forceinline__ double ldv(const UGKS_GLOBAL S* plane, int idx) {
  return (double)ldb(plane, (unsigned)idx * (unsigned)sizeof(S));
}
template <typename S>
__device__ __forceinline__ void stv(UGKS_GLOBAL S* plane, int idx, double x) {
  *reinterpret_cast<UGKS_GLOBAL S*>(reinterpret_cast<UGKS_GLOBAL char*>(plane) +
                                    (unsigned)idx * (unsigned)sizeof(S)) = static_cast<S>(x);
}
template <typename S>
__device__ __forceinline__ const UGKS_GLOBAL S* plane_of(const UGKS_GLOBAL S* f, const KParams& P,
                                                         int p) {
  return f + (long long)p * P.PS;
}
template <typename S>
__device__ __forceinline__ UGKS_GLOBAL S* plane_of(UGKS_GLOBAL S* f, const KParams& P, int p) {
  return f + (long long)p * P.PS;
}
// Buffer resource of one plane (base, size in bytes): loads at a per-lane 32-bit byte offset
// from a scalar base, range-checked by the hardware.  The size field is an unsigned 32-bit
// count (a plane holds at most 2^28 values, so at most 2^31 bytes).  Word 3 selects 32-bit
// data for the untyped buffer instructions.
template <typename S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const UGKS_GLOBAL S* plane,
                                                             const KParams& P) {
  const unsigned bytes = (unsigned)((unsigned long long)P.PS * sizeof(S));
  return __builtin_amdgcn_make_buffer_rsrc((void*)plane, (short)0, __builtin_bit_cast(int, bytes),
                                           0x00020000);
}
// Stores through the same resources; an offset past the plane's range is dropped by the
// hardware range check, so lanes without a cell to write need no branch.
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned off, double x, double) {
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, x), r, off, 0, 0);
}
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned off, double x, float) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)x), r, off, 0, 0);
}
// Loads through the same resources, in the storage type (converted where they are used).
__device__ __forceinline__ double bload_raw(__amdgpu_buffer_rsrc_t r, unsigned off, double) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float bload_raw(__amdgpu_buffer_rsrc_t r, unsigned off, float) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// index of cell (i, j) in a plane; i and j may lie in the halo
__device__ __forceinline__ int pidx(const KParams& P, int i, int j) {
  return (j + kHalo) * P.Lx + i + kHalo;
}

// ------------------------------------------------------------------ lane exchange
// Whole-wavefront DPP shifts by one lane: lane l receives the value lane l - 1 holds
// (from_lower) or lane l + 1 holds (from_upper); the edge lane, which has no source, reads 0
// (bound control), so no copy of an "old" value is needed.
__device__ __forceinline__ double dpp_shift(double x, int ctrl_lower) {
  const long long b = __double_as_longlong(x);
  const int lo = (int)(unsigned)(b & 0xffffffffll), hi = (int)(b >> 32);
  int rlo, rhi;
  if (ctrl_lower) {
    rlo = __builtin_amdgcn_mov_dpp(lo, 0x138, 0xf, 0xf, true);  // wave_shr:1
    rhi = __builtin_amdgcn_mov_dpp(hi, 0x138, 0xf, 0xf, true);
  } else {
    rlo = __builtin_amdgcn_mov_dpp(lo, 0x130, 0xf, 0xf, true);  // wave_shl:1
    rhi = __builtin_amdgcn_mov_dpp(hi, 0x130, 0xf, 0xf, true);
  }
  return __longlong_as_double(((long long)rhi << 32) | (long long)(unsigned)rlo);
}
__device__ __forceinline__ double from_lower(double x) { return dpp_shift(x, 1); }
__device__ __forceinline__ double from_upper(double x) { return dpp_shift(x, 0); }
__device__ __forceinline__ float from_lower(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_upper(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x130, 0xf, 0xf, true));
}

// ------------------------------------------------------------------ pointwise physics
// Reciprocal: the hardware estimate (relative error below 5e-8 on gfx950) refined by one
// Newton step (below 3e-15).
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// Van Leer limited slope of two one-sided differences p, q (second-order reconstruction,
// Sec. 2.A), 2 p q / ((p + q) dx) when p and q agree in sign, else 0, times half a cell: the
// change of the reconstruction from the cell centre to a face, p q / (p + q).
__device__ __forceinline__ double half_limited(double p, double q) {
  const double pq = p * q;
  const double r = pq * recip(p + q);
  return pq > 0.0 ? r : 0.0;
}
// The same, forced to zero where `keep` is false (ghost columns, rows next to a wall): in the
// update kernel the mask joins the sign test instead of multiplying the result (one FP64
// multiply less per limiter; in the moment kernel the multiply measured faster).
__device__ __forceinline__ double half_limited(double p, double q, bool keep) {
  const double pq = p * q;
  const double r = pq * recip(p + q);
  return (pq > 0.0 && keep) ? r : 0.0;
}
// FP32 forms (the FP32-storage update): the hardware reciprocal is accurate to 1 ulp.
__device__ __forceinline__ float half_limited(float p, float q) {
  const float pq = p * q;
  const float r = pq * __builtin_amdgcn_rcpf(p + q);
  return pq > 0.0f ? r : 0.0f;
}
__device__ __forceinline__ float half_limited(float p, float q, bool keep) {
  const float pq = p * q;
  const float r = pq * __builtin_amdgcn_rcpf(p + q);
  return (pq > 0.0f && keep) ? r : 0.0f;
}
__device__ __forceinline__ float exp_of(float x) { return expf(x); }
__device__ __forceinline__ double exp_of(double x) { return exp(x); }
__device__ __forceinline__ float expm1_of(float x) { return expm1f(x); }
__device__ __forceinline__ double expm1_of(double x) { return expm1(x); }


struct Prim {
  double rho, U, V, lam;  // lambda = 1/T
};

// Primitive variables of W = (rho, rho U, rho V, rho E) of a 2D gas with dof internal degrees
// of freedom: rho E = rho (U^2 + V^2)/2 + (2 + dof) rho/(4 lambda), lam_c = (2 + dof)/4 (the
// paper's gas: dof = 0).  false on an invalid state.
template <typename Ptr>
__device__ __forceinline__ bool prim_of(Ptr W, Prim& p, double lam_c) {
  const double rho = W[0];
  const double U = W[1] / rho;
  const double V = W[2] / rho;
  const double e = W[3] - 0.5 * rho * (U * U + V * V);
  p.rho = rho;
  p.U = U;
  p.V = V;
  p.lam = lam_c * rho / e;
  return rho > 0.0 && e > 0.0 && isfinite(rho) && isfinite(e) && isfinite(U) && isfinite(V) &&
         isfinite(p.lam);
}

// BGK collision time tau = mu/p, mu = mu_ref T^(1/2), p = rho T/2.
__device__ __forceinline__ double collision_time(const Prim& p, double mu_ref) {
  return 2.0 * mu_ref * sqrt(p.lam) / p.rho;
}

// Moments 0..6 of the normalised 1D Maxwellian along one axis: full line, and one half of it
// (side 0: u > 0, 1: u < 0), from their first two and the factors c[n] of the recurrence.
__device__ __forceinline__ void axis_factors(double lam, double* c) {
#pragma unroll
  for (int n = 2; n < 7; ++n) c[n] = (double)(n - 1) / (2.0 * lam);
}
__device__ __forceinline__ void axis_full(double U, const double* c, double* m) {
  m[0] = 1.0;
  m[1] = U;
#pragma unroll
  for (int n = 2; n < 7; ++n) m[n] = U * m[n - 1] + c[n] * m[n - 2];
}
__device__ __forceinline__ void axis_half_line(double U, const double* c, double m0, double edge,
                                               int side, double* m) {
  m[0] = m0;
  m[1] = U * m[0] + (side == 0 ? edge : -edge);
#pragma unroll
  for (int n = 2; n < 7; ++n) m[n] = U * m[n - 1] + c[n] * m[n - 2];
}
__device__ __forceinline__ double axis_edge(double U, double lam) {
  return exp(-lam * U * U) / (2.0 * sqrt(kPi * lam));
}
__device__ __forceinline__ double axis_m0(double U, double lam, int side) {
  const double sU = sqrt(lam) * U;
  return 0.5 * erfc(side == 0 ? -sU : sU);
}

// Gaussian moments of the internal coordinates xi at lambda: x2 = <|xi|^2> = dof/(2 lambda),
// x4 = <|xi|^4> = dof (dof + 2)/(4 lambda^2).  They enter through psi_4 = (un^2 + ut^2 + |xi|^2)/2;
// kXi = false is the paper's gas, whose moments carry no xi terms.
struct Xi {
  double x2, x4;
};

// <un^a ut^b psi>, psi = (1, un, ut, psi_4)
template <bool kXi>
__device__ __forceinline__ void mpsi(const double* mu, const double* mv, int a, int b,
                                     const Xi& xi, double* o) {
  o[0] = mu[a] * mv[b];
  o[1] = mu[a + 1] * mv[b];
  o[2] = mu[a] * mv[b + 1];
  if constexpr (kXi)
    o[3] = 0.5 * (mu[a + 2] * mv[b] + mu[a] * mv[b + 2] + xi.x2 * (mu[a] * mv[b]));
  else
    o[3] = 0.5 * (mu[a + 2] * mv[b] + mu[a] * mv[b + 2]);
}

// <un^a ut^b psi (c . psi)>; the |xi|^2 of c_4 psi_4 brings <|xi|^2 un^a ut^b psi>
template <bool kXi>
__device__ __forceinline__ void mpsi_c(const double* mu, const double* mv, int a, int b,
                                       const Xi& xi, const double* c, double* o) {
  double t0[4], t1[4], t2[4], t3[4], t4[4];
  mpsi<kXi>(mu, mv, a, b, xi, t0);
  mpsi<kXi>(mu, mv, a + 1, b, xi, t1);
  mpsi<kXi>(mu, mv, a, b + 1, xi, t2);
  mpsi<kXi>(mu, mv, a + 2, b, xi, t3);
  mpsi<kXi>(mu, mv, a, b + 2, xi, t4);
  if constexpr (kXi) {
    const double m00 = mu[a] * mv[b];
    const double tx[4] = {xi.x2 * m00, xi.x2 * (mu[a + 1] * mv[b]), xi.x2 * (mu[a] * mv[b + 1]),
                          0.5 * (xi.x2 * (mu[a + 2] * mv[b] + mu[a] * mv[b + 2]) + xi.x4 * m00)};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      o[q] = c[0] * t0[q] + c[1] * t1[q] + c[2] * t2[q] + 0.5 * c[3] * (t3[q] + t4[q] + tx[q]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      o[q] = c[0] * t0[q] + c[1] * t1[q] + c[2] * t2[q] + 0.5 * c[3] * (t3[q] + t4[q]);
  }
}

// S4 micro slope: a such that the moments of rho g (a . psi) equal s (closed form, 2D gas with
// q_c = (2 + dof)/2 and a4_c = 4/(2 + dof); the paper's gas has 1 and 2).
__device__ __forceinline__ void micro_slope(const Prim& p, const double* s, double* a,
                                            double q_c, double a4_c) {
  const double q2 = p.U * p.U + p.V * p.V + q_c / p.lam;
  const double R2 = s[1] - p.U * s[0];
  const double R3 = s[2] - p.V * s[0];
  const double R4 = 2.0 * s[3] - q2 * s[0];
  a[3] = a4_c * p.lam * p.lam / p.rho * (R4 - 2.0 * p.U * R2 - 2.0 * p.V * R3);
  a[2] = 2.0 * p.lam * R3 / p.rho - p.V * a[3];
  a[1] = 2.0 * p.lam * R2 / p.rho - p.U * a[3];
  a[0] = s[0] / p.rho - p.U * a[1] - p.V * a[2] - 0.5 * a[3] * q2;
}

// S3 time weights of Eq. (2) integrated over [0, dt]:
// Mt1 int(1 - e^{-t/tau}), Mt2 -int(tau(1 - e^{-t/tau}) - t e^{-t/tau}),
// Mt3 int(t - tau(1 - e^{-t/tau})), Mt4 int e^{-t/tau}, Mt5 int t e^{-t/tau}.
__device__ __forceinline__ void time_weights(double dt, double tau, double* Mt) {
  const double e = exp(-dt / tau);
  Mt[3] = -tau * expm1(-dt / tau);
  Mt[4] = tau * Mt[3] - tau * dt * e;
  Mt[0] = dt - Mt[3];
  Mt[1] = -tau * Mt[0] + Mt[4];
  Mt[2] = 0.5 * dt * dt - tau * Mt[0];
}

// The step of the launch's step (parity = the f/W buffer it reads): fixed, or with the
// adaptive step cfl / rmax of the state W^n it starts from.
__device__ __forceinline__ double step_dt(const KParams& P, int parity) {
  if (!P.adaptive) return P.dt;
  return P.cfl / __longlong_as_double((long long)P.rmax[parity]);
}

// ------------------------------------------------------------------ addressing
__device__ __forceinline__ int wrap(int i, int n) { return ((i % n) + n) % n; }
__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// Plane column that the lane of cell i (which may lie beyond the mesh) loads: a periodic image, or
// in a channel the column itself, of the halo at most.
__device__ __forceinline__ int plane_col(const KParams& P, int i) {
  return P.bc == UGKS_BC_PERIODIC ? wrap(i, P.nx) : (i < P.nx + 1 ? i : P.nx + 1);
}

// Place of the first value of sum q (16: the Shakhov model's heat sum) of face side s, which is one of
// an x (y) face, and of the raw moment r of the Shakhov model's cells, in a chunk's moment sums
// (hs_part).
template <bool kX>
__device__ __forceinline__ long long sum_at(const KParams& P, int s, int q) {
  const int first = q < 16 ? 16 * s + q : s;
  const long long at = kX ? (long long)first * (P.nc + P.ny)
                          : (long long)first * P.nc + (q < 16 ? 32LL : 2LL) * P.ny;
  return q < 16 ? at : at + (long long)kSlotHeat * P.nc + 32LL * P.ny;
}
__device__ __forceinline__ long long cell_sum_at(const KParams& P, int r) {
  return (long long)(kSlotCell + r) * P.nc + 34LL * P.ny;
}

// Workgroups are handed to the 8 XCDs round-robin; renumber the n of one instance so that each XCD
// works through one contiguous range of them (its own L2 then serves the rows its neighbours also
// read) and all XCDs work on every instance.  Which XCD its first block falls on does not matter:
// blocks 8 apart share one.  (With every instance filled up to a multiple of 8 blocks, a step of 256
// solves of 4..8 x 3..6 cells at 8^2 took 149 us, without 107; of 16 periodic ones of 60..135 x
// 20..35 cells at 24..32 x 24 404 and 367.)
constexpr int kXcd = 8;
__device__ __forceinline__ int xcd_block(int local, int n) {
  const int q = n / kXcd, r = n % kXcd, x = local % kXcd, i = local / kXcd;
  return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// ------------------------------------------------------------------ wave reductions
__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1) x = fmax(x, __shfl_xor(x, h, kWave));
  return x;
}

// Node range of one half of a velocity axis.  Half s = +1 takes the nodes with positive
// velocity, s = -1 the negative ones; a node at exactly zero belongs to both halves when
// `share_zero` (moment sums, each visit with weight 1/2), else only to the positive half.
struct Half {
  int first, count, step;
};
__device__ __forceinline__ Half axis_half(int n, int s, bool share_zero) {
  const int odd = n & 1, mid = n >> 1;  // with n odd, node mid is zero
  Half h;
  if (s > 0) {
    h.first = mid;
    h.count = n - mid;
    h.step = 1;
  } else {
    h.first = mid - 1 + (share_zero ? odd : 0);
    h.count = h.first + 1;
    h.step = -1;
  }
  return h;
}

// Nodes [a0, a1) of a half's node sequence taken by velocity chunk g of G.
__host__ __device__ __forceinline__ void chunk_range(int count, int g, int G, int& a0, int& a1) {
  a0 = (int)((long long)g * count / G);
  a1 = (int)((long long)(g + 1) * count / G);
}

// Workgroup L of a cell kernel: row segment t (fastest), row j, velocity chunk g.  The
// workgroups an XCD runs at once then cover whole rows of a band of neighbouring rows, so the
// cache lines a segment shares with the next one, and the rows j +- 1, j +- 2 it reads, come
// from that XCD's L2.
__device__ __forceinline__ void cell_block(int L, int ny, int ntx, int& t, int& g, int& j) {
  t = L % ntx;
  const int r = L / ntx;
  j = r % ny;
  g = r / ny;
}

// ------------------------------------------------------------------ launch plans
typedef const Inst* __restrict__ inst_cptr;
typedef const int* __restrict__ int_cptr;

// Instance owning workgroup b: the last instance whose first workgroup is <= b (uniform).
__device__ __forceinline__ int find_inst(const int* off_generic, int n, int b) {
  const int_cptr off = (int_cptr)off_generic;
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= b)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int first_block(const int* off_generic, int ii) {
  return ((int_cptr)off_generic)[ii];
}

// The kernels of a step take the members of the plan view that they need one by one (inst, the
// offsets of their workgroups off, ninst, step): such arguments come in scalar registers with the
// wavefront (-amdgpu-kernarg-preload-count), where a structure is read from memory, 0.4 us at the
// start of every launch (a step of 40 x 10 cells 28.2 -> 27.6 us).  The plan is read-only for the
// whole launch.

// ================================================================== kernels
// Discrete Maxwellian of each cell's W (initial state), one thread per plane value; the
// planes of H hold dof/(2 lambda) times those of G.
template <typename S>
__global__ __launch_bounds__(256) void init_kernel(PlanView pv) {
  const Inst* __restrict__ I = pv.inst;
  const KParams P = I->P;
  UGKS_GLOBAL S* f = static_cast<UGKS_GLOBAL S*>(I->f[I->cur]);
  const UGKS_GLOBAL double* W = I->W[I->cur];
  const long long nc = (long long)P.nx * P.ny;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nc * P.NV * P.NC) return;
  const int p = (int)(e / nc);
  const int c = (int)(e - (long long)p * nc);
  const int j = c / P.nx, i = c - j * P.nx;
  Prim pr;
  if (!prim_of(W + 4 * (size_t)c, pr, P.lam_c) && p == 0) *P.flag = 1;
  const bool h = p >= P.NV;
  const int pg = h ? p - P.NV : p;
  const int k = pg / P.M, m = pg - k * P.M;
  const double du = P.uk[k] - pr.U, dv = P.vm[m] - pr.V;
  double g = pr.rho * pr.lam / kPi * exp(-pr.lam * (du * du + dv * dv));
  if (h) g *= (double)P.dof / (2.0 * pr.lam);
  stv(plane_of(f, P, p), pidx(P, i, j), g);
}

// Debug: quiet NaN in every cell value of the f and W buffers the next step writes (the
// halo is left as it is: the kernels read it, where a wall or ghost switch discards it).  A
// step that failed to write one of these values would leave a NaN in the state.
template <typename S>
__global__ __launch_bounds__(256) void poison_kernel(PlanView pv) {
  const Inst* __restrict__ I = pv.inst;
  const KParams P = I->P;
  const int nxt = (I->cur + pv.step + 1) & 1;
  UGKS_GLOBAL S* f = static_cast<UGKS_GLOBAL S*>(I->f[nxt]);
  UGKS_GLOBAL double* W = I->W[nxt];
  const long long nc = (long long)P.nx * P.ny;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nc * P.NV * P.NC) return;
  const int p = (int)(e / nc);
  const int c = (int)(e - (long long)p * nc);
  const int j = c / P.nx, i = c - j * P.nx;
  plane_of(f, P, p)[pidx(P, i, j)] = static_cast<S>(__builtin_nan(""));
  // a channel's ghost columns, which the update kernel writes into f^{n+1}
  if (P.bc == UGKS_BC_CHANNEL && (i == 0 || i == P.nx - 1))
    plane_of(f, P, p)[pidx(P, i == 0 ? -1 : P.nx, j)] = static_cast<S>(__builtin_nan(""));
  if (p == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) W[4 * (size_t)c + q] = __builtin_nan("");
  }
}

// Ghost state of row j of a channel (Sec. 3.A) from the primitive state pc of the cell next
// to it: the inlet (side 0) holds p_in and T_in (its velocity that of the cell, or the fixed
// inlet profile), the outlet (side 1) p_out with the cell's velocity and temperature.
__device__ __forceinline__ Prim ghost_prim(const KParams& P, int side, int j, const Prim& pc) {
  Prim pg;
  if (side == 0) {
    const double T = P.T_in;
    pg.lam = 1.0 / T;
    pg.rho = 2.0 * P.p_in / T;
    if (P.inlet_fixed_u) {
      pg.U = P.U_in * (1.0 + P.U_noise * P.xi_in[j]);
      pg.V = 0.0;
    } else {
      pg.U = pc.U;
      pg.V = pc.V;
    }
  } else {
    const double T = 1.0 / pc.lam;
    pg.rho = 2.0 * P.p_out / T;
    pg.U = pc.U;
    pg.V = pc.V;
    pg.lam = pc.lam;
  }
  return pg;
}

// Ghost state W of a channel ghost cell, stored for the interface kernel.
__device__ __forceinline__ void store_wg(UGKS_GLOBAL double* wg, const Prim& pg, double lam_c) {
  wg[0] = pg.rho;
  wg[1] = pg.rho * pg.U;
  wg[2] = pg.rho * pg.V;
  wg[3] = 0.5 * pg.rho * (pg.U * pg.U + pg.V * pg.V) + lam_c * pg.rho / pg.lam;
}

// Halo rows of the current f of a periodic box (a step's first launch): the two rows below and
// above the mesh of every plane take the periodic images, one thread per value.  The columns need
// no halo: the cell kernels' lanes beyond the mesh load the images themselves (plane_col).  With
// the columns copied too, eight scattered bytes at a time, 96 x 80 cells at 33^2 took 100.7 us a
// step, without them 99.0.  A channel's halo is written by the update kernel (its ghost columns; the
// rest stays zero).
constexpr int kGhostThreads = 256;
__host__ __device__ __forceinline__ int ghost_blocks(int nx) {
  return (2 * kHalo * nx + kGhostThreads - 1) / kGhostThreads;  // of one plane
}
template <typename S>
__global__ __launch_bounds__(kGhostThreads) void ghost_kernel(const Inst* inst,
                                                              const int* off, int ninst,
                                                              int step) {
  const int b = blockIdx.x;
  const int ii = find_inst(off, ninst, b);
  const Inst* __restrict__ I = inst + ii;
  const KParams P = I->P;
  UGKS_GLOBAL S* f = static_cast<UGKS_GLOBAL S*>(I->f[(I->cur + step) & 1]);
  const int local = b - first_block(off, ii);
  const int bpp = ghost_blocks(P.nx);
  const int p = local / bpp;
  const int e = (local - p * bpp) * kGhostThreads + threadIdx.x;
  const int r = e / P.nx, i = e - r * P.nx;
  if (r >= 2 * kHalo) return;
  const int j = r < kHalo ? r - kHalo : P.ny + r - kHalo;
  UGKS_GLOBAL S* pl = plane_of(f, P, p);
  stv(pl, pidx(P, i, j), ldv(pl, pidx(P, i, wrap(j, P.ny))));
}

// Per cell: slopes and the outgoing moment sums of all four faces.  A workgroup takes one
// segment of kTileS cells of one row (lanes hold the segment and one neighbour on each side);
// wavefront q sums velocity quadrant q into the x face and the y face its particles leave
// through.  Along one v line (u fixed) every sum is a combination of the running v moments
//   F^n = sum_m w_m v^n f,  X^n = sum_m w_m v^n hx,  Y^n = sum_m w_m v^n hy
// (hx, hy: half-cell changes; n up to 3, 3 and 4), with f_hat = f + s hx (or s hy) and
// D = (2u/dx) hx + (2v/dy) hy; the 32 face sums take them in once per line.  The two partial
// sums of each face side meet in LDS at the end.  With internal degrees of freedom the
// chunks G..2G-1 of a segment walk the planes of H, whose psi is (0, 0, 0, 1/2): they add to
// the energy sums only.  The Shakhov instantiation (kShak) also sums, per face side, ut c2h
// of the reconstruction (c2h = (un^2 + ut^2)/2) and, per cell, eight raw moments of f for
// the heat fluxes.
template <typename S, bool kShak>
__global__ __launch_bounds__(kWave* kQuads) void sums_kernel(const Inst* inst, const int* off,
                                                               int ninst, int step) {
  constexpr int kR = kShak ? 17 : 16;
  __shared__ double red[4][kR][kWave];
  __shared__ double cellred[kShak ? 3 : 1][8][kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ii = find_inst(off, ninst, blockIdx.x);
  const Inst* __restrict__ I = inst + ii;
  const KParams P = I->P;
  const int G = I->gsplit;
  const int ntx = (P.nx + kTileS - 1) / kTileS;
  const int b = xcd_block(blockIdx.x - first_block(off, ii), ntx * P.ny * G * P.NC);
  int t, gg, j;
  cell_block(b, P.ny, ntx, t, gg, j);
  const bool hpart = gg >= G;  // planes of H
  const int g = hpart ? gg - G : gg;
  const UGKS_GLOBAL S* f = static_cast<const UGKS_GLOBAL S*>(I->f[(I->cur + step) & 1]) +
                           (hpart ? (long long)P.NV * P.PS : 0ll);
  UGKS_GLOBAL double* hs = I->hs + gg * P.part;
  const int i = t * kTileS - 1 + lane;
  const bool valid = lane >= 1 && lane <= kTileS && i < P.nx;
  // channel ghost columns (i = -1, nx): their sums towards the domain are the ghost sums of
  // the inlet and outlet faces (zero slopes); only the first and last segments hold them
  const bool chan = P.bc == UGKS_BC_CHANNEL;
  const bool ghost = chan && (i == -1 || i == P.nx);
  const bool ghost_wave = chan && (t == 0 || (t + 1) * kTileS >= P.nx);
  const int o = pidx(P, plane_col(P, i), j);
  const unsigned bs = (unsigned)sizeof(S);
  const unsigned oc = (unsigned)o * bs, oS = (unsigned)(o - P.Lx) * bs;
  const unsigned oN = (unsigned)(o + P.Lx) * bs;
  const double my = (P.bc == UGKS_BC_CHANNEL && (j == 0 || j == P.ny - 1)) ? 0.0 : 1.0;
  const int su = quad_su(q), sv = quad_sv(q);
  // each half is walked inwards, towards v = 0 and u = 0: the update kernel walks it
  // outwards, so each kernel starts on the planes the other touched last
  const Half hu0 = axis_half(P.K, su, true), hv0 = axis_half(P.M, sv, true);
  const Half hu = {hu0.first + (hu0.count - 1) * hu0.step, hu0.count, -hu0.step};
  const Half hv = {hv0.first + (hv0.count - 1) * hv0.step, hv0.count, -hv0.step};
  const double two_idx = 2.0 * P.inv_dx, two_idy = 2.0 * P.inv_dy;
  double ax[kR], ay[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) ax[r] = ay[r] = 0.0;
  // raw cell moments (kShak): f, u f, v f, u^2 f, u v f, v^2 f, u |c|^2 f, v |c|^2 f
  double cm[kShak ? 8 : 1];
#pragma unroll
  for (int r = 0; r < (kShak ? 8 : 1); ++r) cm[r] = 0.0;
  int a0, a1;
  chunk_range(hu.count, g, G, a0, a1);
  // The wavefronts of a SIMD are issued oldest first, so the later ones fall behind and end alone.
  // Here a wavefront is issued before those that are a quarter of their lines further on: FP32
  // storage at 400 x 100 x 40^2 113 -> 109 us, FP64 Shakhov at 130 x 37 x 40^2 34.9 -> 33.4.  FP64
  // BGK, which waits for its loads more than for issue, is slower with it (190 -> 196 us).  It costs
  // registers: the FP32 BGK form then takes 151, three waves per SIMD instead of four, and held to
  // four it spills and takes 117 us; the FP32 Shakhov form would take 171 instead of 165, two waves
  // instead of three (400 x 100 x 40^2 115 -> 154 us), so it goes without.
  constexpr bool kEven = (sizeof(S) == 4) != kShak;
  for (int a = a0; a < a1; ++a) {
    if constexpr (kEven) {
      const int done = 4 * (a - a0);
      if (done < a1 - a0)
        __builtin_amdgcn_s_setprio(3);
      else if (done < 2 * (a1 - a0))
        __builtin_amdgcn_s_setprio(2);
      else if (done < 3 * (a1 - a0))
        __builtin_amdgcn_s_setprio(1);
      else
        __builtin_amdgcn_s_setprio(0);
    }
    const int k = hu.first + a * hu.step;
    const double u = P.uk[k];
    const double wu = P.wk[k] * (u == 0.0 ? 0.5 : 1.0);
    const UGKS_GLOBAL S* line = plane_of(f, P, k * P.M);
    double F0 = 0, F1 = 0, F2 = 0, F3 = 0, X0 = 0, X1 = 0, X2 = 0, X3 = 0;
    double Y0 = 0, Y1 = 0, Y2 = 0, Y3 = 0, Y4 = 0;
    struct Vals {
      S c, s, n;  // in the storage type
    };
    // planes and weight rows are walked with running pointers: one add per node each
    const long long pstep = (long long)hv.step * P.PS;
    const UGKS_GLOBAL S* pcur = line + (long long)hv.first * P.PS;
    const UGKS_CONST double* wp = (const UGKS_CONST double*)(P.vmom + 5 * hv.first);
    // FP64: each node's weights are requested one node ahead, as scalar loads (one node
    // beyond the last node of a half lies in the other half)
    double w0 = wp[0], w1 = wp[1], w2 = wp[2], w3 = wp[3], w4 = wp[4];
    const int wstep = 5 * hv.step;
    auto load_at = [&](const UGKS_GLOBAL S* p) {
      const __amdgpu_buffer_rsrc_t r = plane_rsrc(p, P);
      return Vals{bload_raw(r, oc, S{}), bload_raw(r, oS, S{}), bload_raw(r, oN, S{})};
    };
    auto node = [&](const Vals& x) {
      // w_m v_m^n, n = 0..4, with the weight 1/2 of a node at v = 0 (visited by both halves)
      double n0 = 0.0, n1 = 0.0, n2 = 0.0, n3 = 0.0, n4 = 0.0;
      if constexpr (sizeof(S) == 8) {
        n0 = wp[wstep];
        n1 = wp[wstep + 1];
        n2 = wp[wstep + 2];
        n3 = wp[wstep + 3];
        n4 = wp[wstep + 4];
      } else {  // FP32 storage: read at the node (with the next node's held, 600 x 300 x 24^2 took
                // 195 us instead of 191, 120 x 60 x 29^2 20.5 instead of 20.0)
        w0 = wp[0];
        w1 = wp[1];
        w2 = wp[2];
        w3 = wp[3];
        w4 = wp[4];
      }
      // slopes in the storage type (FP32 storage: FP32 slopes), sums in FP64
      const S fW = from_lower(x.c), fE = from_upper(x.c);
      const double hx = half_limited(fE - x.c, x.c - fW);
      const double hy = my * (double)half_limited(x.n - x.c, x.c - x.s);
      const double fc = x.c;
      F0 = fma(fc, w0, F0);
      F1 = fma(fc, w1, F1);
      F2 = fma(fc, w2, F2);
      F3 = fma(fc, w3, F3);
      X0 = fma(hx, w0, X0);
      X1 = fma(hx, w1, X1);
      X2 = fma(hx, w2, X2);
      X3 = fma(hx, w3, X3);
      Y0 = fma(hy, w0, Y0);
      Y1 = fma(hy, w1, Y1);
      Y2 = fma(hy, w2, Y2);
      Y3 = fma(hy, w3, Y3);
      Y4 = fma(hy, w4, Y4);
      wp += wstep;
      if constexpr (sizeof(S) == 8) {
        w0 = n0;
        w1 = n1;
        w2 = n2;
        w3 = n3;
        w4 = n4;
      }
    };
    if constexpr (sizeof(S) == 8) {
      // FP64: two value sets, each node's loads issued one node ahead (deeper prefetch costs
      // this kernel its fourth wave per SIMD)
      Vals va = load_at(pcur);
      int c = 0;
      for (; c + 1 < hv.count; c += 2) {
        pcur += pstep;
        const Vals vb = load_at(pcur);
        node(va);
        if (c + 2 < hv.count) pcur += pstep;
        va = load_at(pcur);
        node(vb);
      }
      if (c < hv.count) node(va);
    } else {
      // FP32 storage: a row load brings half the bytes, so each node's loads are issued six
      // nodes ahead (kSA + 1 value sets in a ring; 3 and 4 ahead measured 6% and 2% slower at
      // 400 x 100 x 40^2); past the last node of the half the loads read its plane again
      constexpr int kSA = 6, NB = kSA + 1;
      int nl = 0;
      auto load_next = [&]() {
        const Vals v = load_at(pcur);
        if (++nl < hv.count) pcur += pstep;
        return v;
      };
      Vals ring[NB];
#pragma unroll
      for (int d = 0; d < kSA; ++d) ring[d] = load_next();
      int c = 0;
      for (; c + NB <= hv.count; c += NB) {
#pragma unroll
        for (int s = 0; s < NB; ++s) {
          ring[(s + kSA) % NB] = load_next();
          node(ring[s]);
        }
      }
#pragma unroll
      for (int s = 0; s < NB; ++s) {
        if (c + s < hv.count) {
          ring[(s + kSA) % NB] = load_next();
          node(ring[s]);
        }
      }
    }
    if (ghost_wave && ghost) {  // a ghost cell has zero slopes
      X0 = X1 = X2 = X3 = 0.0;
      Y0 = Y1 = Y2 = Y3 = Y4 = 0.0;
    }
    // moments of the x-face reconstruction (S), the y-face one (R) and of D
    const double ucx = u * two_idx, u2h = 0.5 * u * u, wuu = wu * u;
    if (hpart) {
      const double wh = 0.5 * wu, whu = 0.5 * wuu;
      const double S0 = su > 0 ? F0 + X0 : F0 - X0;
      const double R0 = sv > 0 ? F0 + Y0 : F0 - Y0, R1 = sv > 0 ? F1 + Y1 : F1 - Y1;
      const double D0 = fma(ucx, X0, two_idy * Y1), D1 = fma(ucx, X1, two_idy * Y2);
      ax[3] = fma(wh, S0, ax[3]);
      ax[7] = fma(wh, Y0, ax[7]);
      ax[11] = fma(whu, S0, ax[11]);
      ax[15] = fma(whu, D0, ax[15]);
      ay[3] = fma(wh, R0, ay[3]);
      ay[7] = fma(wh, X0, ay[7]);
      ay[11] = fma(wh, R1, ay[11]);
      ay[15] = fma(wh, D1, ay[15]);
      continue;
    }
    const double S0 = su > 0 ? F0 + X0 : F0 - X0, S1 = su > 0 ? F1 + X1 : F1 - X1;
    const double S2 = su > 0 ? F2 + X2 : F2 - X2;
    const double R0 = sv > 0 ? F0 + Y0 : F0 - Y0, R1 = sv > 0 ? F1 + Y1 : F1 - Y1;
    const double R2 = sv > 0 ? F2 + Y2 : F2 - Y2, R3 = sv > 0 ? F3 + Y3 : F3 - Y3;
    const double D0 = fma(ucx, X0, two_idy * Y1), D1 = fma(ucx, X1, two_idy * Y2);
    const double D2 = fma(ucx, X2, two_idy * Y3), D3 = fma(ucx, X3, two_idy * Y4);
    // x face: psi = (1, u, v, c2h), c2h = (u^2 + v^2)/2
    const double cS = fma(u2h, S0, 0.5 * S2), cT = fma(u2h, Y0, 0.5 * Y2);
    const double cD = fma(u2h, D0, 0.5 * D2);
    ax[0] = fma(wu, S0, ax[0]);
    ax[1] = fma(wuu, S0, ax[1]);
    ax[2] = fma(wu, S1, ax[2]);
    ax[3] = fma(wu, cS, ax[3]);
    ax[4] = fma(wu, Y0, ax[4]);
    ax[5] = fma(wuu, Y0, ax[5]);
    ax[6] = fma(wu, Y1, ax[6]);
    ax[7] = fma(wu, cT, ax[7]);
    ax[8] = fma(wuu, S0, ax[8]);
    ax[9] = fma(wuu * u, S0, ax[9]);
    ax[10] = fma(wuu, S1, ax[10]);
    ax[11] = fma(wuu, cS, ax[11]);
    ax[12] = fma(wuu, D0, ax[12]);
    ax[13] = fma(wuu * u, D0, ax[13]);
    ax[14] = fma(wuu, D1, ax[14]);
    ax[15] = fma(wuu, cD, ax[15]);
    // y face: psi = (1, v, u, c2h)
    const double cR = fma(u2h, R0, 0.5 * R2), cX = fma(u2h, X0, 0.5 * X2);
    const double cR1 = fma(u2h, R1, 0.5 * R3), cD1 = fma(u2h, D1, 0.5 * D3);
    ay[0] = fma(wu, R0, ay[0]);
    ay[1] = fma(wu, R1, ay[1]);
    ay[2] = fma(wuu, R0, ay[2]);
    ay[3] = fma(wu, cR, ay[3]);
    ay[4] = fma(wu, X0, ay[4]);
    ay[5] = fma(wu, X1, ay[5]);
    ay[6] = fma(wuu, X0, ay[6]);
    ay[7] = fma(wu, cX, ay[7]);
    ay[8] = fma(wu, R1, ay[8]);
    ay[9] = fma(wu, R2, ay[9]);
    ay[10] = fma(wuu, R1, ay[10]);
    ay[11] = fma(wu, cR1, ay[11]);
    ay[12] = fma(wu, D1, ay[12]);
    ay[13] = fma(wu, D2, ay[13]);
    ay[14] = fma(wuu, D1, ay[14]);
    ay[15] = fma(wu, cD1, ay[15]);
    if constexpr (kShak) {
      const double S3 = su > 0 ? F3 + X3 : F3 - X3;
      ax[16] = fma(wu, fma(u2h, S1, 0.5 * S3), ax[16]);
      ay[16] = fma(wuu, cR, ay[16]);
      const double wu2 = wuu * u;
      cm[0] = fma(wu, F0, cm[0]);
      cm[1] = fma(wuu, F0, cm[1]);
      cm[2] = fma(wu, F1, cm[2]);
      cm[3] = fma(wu2, F0, cm[3]);
      cm[4] = fma(wuu, F1, cm[4]);
      cm[5] = fma(wu, F2, cm[5]);
      cm[6] = fma(wuu, fma(u * u, F0, F2), cm[6]);
      cm[7] = fma(wu, fma(u * u, F1, F3), cm[7]);
    }
  }
  // x faces: (+) from waves 0 and 3, (-) from 1 and 2; y faces: (+) from 0 and 1, (-) from
  // 2 and 3.  Waves 1 and 3 hand their sums over, waves 0 and 2 add and write.
  if (q == 1 || q == 3) {
    const int s = q == 1 ? 0 : 1;
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      red[s][r][lane] = ay[r];
      red[2 + s][r][lane] = ax[r];
    }
  }
  if constexpr (kShak) {
    // every quadrant holds part of each cell's moments; wavefront 0 adds them
    if (q > 0) {
#pragma unroll
      for (int r = 0; r < 8; ++r) cellred[q - 1][r][lane] = cm[r];
    }
  }
  __syncthreads();
  // the inlet ghost's sums towards +x (waves 0 and 3), the outlet ghost's towards -x (waves
  // 1 and 2)
  if (ghost_wave && ghost && q == (i < 0 ? 0 : 2)) {
    const int ox = q == 0 ? 3 : 2, fx = q == 0 ? S_XP : S_XM;
    const size_t cell = (size_t)P.nc + j;
#pragma unroll
    for (int r = 0; r < kR; ++r) hs[sum_at<true>(P, fx, r) + cell] = ax[r] + red[ox][r][lane];
  }
  if (valid && (q == 0 || q == 2)) {
    const size_t cell = (size_t)j * P.nx + i;
    const int fy = q == 0 ? S_YP : S_YM, fx = q == 0 ? S_XP : S_XM;
    const int oy = q == 0 ? 0 : 1, ox = q == 0 ? 3 : 2;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double sx = (ax[r] + red[ox][r][lane]) * (r >= 4 && r < 8 ? two_idy : 1.0);
      const double sy = (ay[r] + red[oy][r][lane]) * (r >= 4 && r < 8 ? two_idx : 1.0);
      hs[sum_at<true>(P, fx, r) + cell] = sx;
      hs[sum_at<false>(P, fy, r) + cell] = sy;
    }
    if constexpr (kShak) {
      hs[sum_at<true>(P, fx, 16) + cell] = ax[16] + red[ox][16][lane];
      hs[sum_at<false>(P, fy, 16) + cell] = ay[16] + red[oy][16][lane];
      if (q == 0) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          hs[cell_sum_at(P, r) + cell] =
              ((cm[r] + cellred[0][r][lane]) + cellred[1][r][lane]) + cellred[2][r][lane];
      }
    }
  }
}

// Heat flux q = sum w c |c|^2 f / 2 about (U, V) from raw sums of f: m0 = sum f, mn = sum un f,
// mt = sum ut f, mnn, mnt, mtt = sum un^2 f, un ut f, ut^2 f, Kn = sum un |c|^2 f,
// Kt = sum ut |c|^2 f, K0 = sum |c|^2 f (|c|^2 = un^2 + ut^2).
__device__ __forceinline__ void heat_flux(double m0, double mn, double mt, double mnn,
                                          double mnt, double mtt, double Kn, double Kt,
                                          double K0, double U, double V, double* q) {
  const double UV2 = U * U + V * V;
  const double c2 = K0 - 2.0 * (U * mn + V * mt) + UV2 * m0;  // sum |u - U|^2 f
  q[0] = 0.5 * (Kn - 2.0 * (U * mnn + V * mnt) + UV2 * mn - U * c2);
  q[1] = 0.5 * (Kt - 2.0 * (U * mnt + V * mtt) + UV2 * mt - V * c2);
}

// Shakhov term of an interface: g0 S0 held over the step adds Mt1 g0 S0 to the distribution
// flux, S0 = k (c . q)(2 lambda |c|^2 - 4), k = (1 - Pr) lambda^2/rho, c = (un - U, ut - V);
// expanded in the record's basis {1, un, ut, c2h, un^2, un ut, ut^2, un c2h, ut c2h} it adds
// to every coefficient of both upwind sides.
// Face records are stored field-major: field f of face e of a family of nf faces (the x faces,
// or the y faces) at f nf + e, so that a wavefront's 64 neighbouring faces read or write one
// field as one contiguous access.  RecRef is one face's record in that layout.
struct RecRef {
  UGKS_GLOBAL double* p;  // field 0 of the face
  size_t nf;              // faces of the family: the stride between fields
  __device__ __forceinline__ UGKS_GLOBAL double& operator[](int f) const {
    return p[(size_t)f * nf];
  }
};

__device__ __forceinline__ void fold_shakhov(double* e, const Prim& p0,
                                             const double* q, double km) {
  const double lam = p0.lam, U = p0.U, V = p0.V;
  const double Q0 = q[0] * U + q[1] * V;
  const double C0 = 2.0 * lam * (U * U + V * V) - 4.0;
  const double l4 = 4.0 * lam;
  const double d[9] = {-C0 * Q0,          l4 * U * Q0 + C0 * q[0], l4 * V * Q0 + C0 * q[1],
                       -l4 * Q0,          -l4 * U * q[0],          -l4 * (V * q[0] + U * q[1]),
                       -l4 * V * q[1],    l4 * q[0],               l4 * q[1]};
#pragma unroll
  for (int n = 0; n < 9; ++n) e[n] = fma(km, d[n], e[n]);
  e[9] = fma(km, d[1], e[9]);
  e[10] = fma(km, d[4], e[10]);
  e[11] = fma(km, d[5], e[11]);
  e[12] = fma(km, d[7], e[12]);
}

// A face of a collisionless gas: free transport alone.
__device__ __forceinline__ void free_flux(double dt, const double* Q1, const double* Q2, double len,
                                          int NC, double* F, RecRef rec, RecRef recH) {
  const double Mt4 = dt, Mt5 = 0.5 * dt * dt;
#pragma unroll
  for (int q = 0; q < 4; ++q) F[q] = len * (Mt4 * Q1[q] - Mt5 * Q2[q]);
  for (int c = 0; c < NC; ++c) {
    const RecRef r = c ? recH : rec;
#pragma unroll
    for (int q = 0; q < 13; ++q) r[R_E + q] = 0.0;
    r[R_GC] = 0.0;
    r[R_LAM] = 0.0;
    r[R_M4] = len * Mt4;
    r[R_M5] = len * Mt5;
    r[R_KIND] = K_FREE;
  }
}

template <bool kXi>
__device__ __forceinline__ Xi xi_of(const KParams& P, const Prim& p0) {
  Xi xi{0.0, 0.0};
  if constexpr (kXi) {
    xi.x2 = (double)P.dof / (2.0 * p0.lam);
    xi.x4 = (double)(P.dof * (P.dof + 2)) / (4.0 * p0.lam * p0.lam);
  }
  return xi;
}

// Shakhov: heat flux of the reconstruction at the interface (local frame); T3 is the sum of
// ut c2h f_hat, the other raw sums are W0 and Q1.
__device__ __forceinline__ void face_heat(const KParams& P, const Prim& p0, const double* W0,
                                          const double* Q1, double T3, double* qh) {
  qh[0] = qh[1] = 0.0;
  if (P.shak)
    heat_flux(W0[0], W0[1], W0[2], Q1[1], Q1[2], 2.0 * W0[3] - Q1[1], 2.0 * Q1[3], 2.0 * T3,
              2.0 * W0[3], p0.U, p0.V, qh);
}

// The macroscopic flux of an interior face: its equilibrium part from the moments e0 .. eA of
// u g0, of its slopes on both sides and in time, and of A; free transport from Q1 and Q2.
__device__ __forceinline__ void macro_flux(const KParams& P, const Prim& p0, const double* Mt,
                                           const double* e0, const double* eL, const double* eR,
                                           const double* eb, const double* eA, const double* Q1,
                                           const double* Q2, const double* qh, double len,
                                           double* F) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    double feq = p0.rho * (Mt[0] * e0[q] + Mt[1] * (eL[q] + eR[q] + eb[q]) + Mt[2] * eA[q]);
    if (q == 3 && P.shak) feq = fma(Mt[0] * P.pr_c, qh[0], feq);
    F[q] = len * (feq + Mt[3] * Q1[q] - Mt[4] * Q2[q]);
  }
}

// The folded polynomial of the equilibrium part of the distribution flux of G, or of H (kXi), and
// what else of the record does not depend on the macroscopic flux.  It is formed in registers and
// stored once: stored and read back to be folded further, the two records of a face took 7 us of
// the interface kernel of 100 x 25 cells, and 3 with the Shakhov model (130 x 37). Averaged over
// xi, the energy term c_4 psi_4 of a slope c contributes c_4 (un^2 + ut^2 + s)/2 to the polynomial
// of G with s = <|xi|^2> = x2, and to that of H, whose Maxwellian is x2 times that of G, with s =
// <|xi|^4>/<|xi|^2> = x4/x2: the constant shifts e0, e1 and e2 by c_4 s/2.
template <bool kXi>
__device__ __forceinline__ void fold_record(const KParams& P, const Prim& p0, const Xi& xi,
                                            const double* Mt, const double* aL,
                                            const double* aR, const double* b,
                                            const double* A, const double* qh, double len,
                                            bool h, RecRef rec) {
  double e[13] = {Mt[0] + Mt[2] * A[0],
                  Mt[1] * aL[0] + Mt[2] * A[1],
                  Mt[1] * b[0] + Mt[2] * A[2],
                  Mt[2] * A[3],
                  Mt[1] * aL[1],
                  Mt[1] * (aL[2] + b[1]),
                  Mt[1] * b[2],
                  Mt[1] * aL[3],
                  Mt[1] * b[3],
                  // R_ER
                  Mt[1] * aR[0] + Mt[2] * A[1],
                  Mt[1] * aR[1],
                  Mt[1] * (aR[2] + b[1]),
                  Mt[1] * aR[3]};
  if (P.shak) fold_shakhov(e, p0, qh, Mt[0] * P.pr_c * p0.lam * p0.lam / p0.rho);
  double gc = len * p0.rho * p0.lam / kPi;
  if constexpr (kXi) {
    const double sc = h ? 0.5 * xi.x4 / xi.x2 : 0.5 * xi.x2;
    e[0] = fma(sc, e[3], e[0]);
    e[1] = fma(sc, e[7], e[1]);
    e[2] = fma(sc, e[8], e[2]);
    e[9] = fma(sc, e[12], e[9]);
    if (h) gc *= xi.x2;
  }
#pragma unroll
  for (int q = 0; q < 13; ++q) rec[R_E + q] = e[q];
  rec[R_GC] = gc;
  rec[R_LAM] = p0.lam;
  rec[R_M4] = len * Mt[3];
  rec[R_M5] = len * Mt[4];
  rec[R_KIND] = K_INTERIOR;
}

// S2-S5 at one interior interface, local frame (internal degrees of freedom: faces_staged).
// S = [W0, Wt, Q1, Q2].  Writes the local macroscopic flux to F, the folded coefficients of the
// distribution flux to rec.
__device__ __forceinline__ void interface_scalars(const KParams& P, double dt, const double* S,
                                                  const double* WL, const double* WR, double dn,
                                                  double len, double* F, RecRef rec, double& U0,
                                                  double& V0, double T3) {
  const double* W0 = S;
  const double* Wt = S + 4;
  const double* Q1 = S + 8;
  const double* Q2 = S + 12;
  Prim p0;
  if (!prim_of(W0, p0, P.lam_c)) *P.flag = 1;
  const Xi xi{0.0, 0.0};
  double Mt[5];
  time_weights(dt, collision_time(p0, P.mu_ref), Mt);
  double swL[4], swR[4], aL[4], aR[4], b[4], A[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    swL[q] = (W0[q] - WL[q]) / (0.5 * dn);
    swR[q] = (WR[q] - W0[q]) / (0.5 * dn);
  }
  micro_slope(p0, swL, aL, P.q_c, P.a4_c);
  micro_slope(p0, swR, aR, P.q_c, P.a4_c);
  micro_slope(p0, Wt, b, P.q_c, P.a4_c);
  double c[7], mu[7], mp[7], mn[7], mv[7];
  axis_factors(p0.lam, c);
  const double edge = axis_edge(p0.U, p0.lam);
  axis_full(p0.U, c, mu);
  axis_half_line(p0.U, c, axis_m0(p0.U, p0.lam, 0), edge, 0, mp);
  axis_half_line(p0.U, c, axis_m0(p0.U, p0.lam, 1), edge, 1, mn);
  axis_full(p0.V, c, mv);
  double m1[4], m2[4], m3[4], sA[4];
  mpsi_c<false>(mp, mv, 1, 0, xi, aL, m1);
  mpsi_c<false>(mn, mv, 1, 0, xi, aR, m2);
  mpsi_c<false>(mu, mv, 0, 1, xi, b, m3);
#pragma unroll
  for (int q = 0; q < 4; ++q) sA[q] = -p0.rho * (m1[q] + m2[q] + m3[q]);
  micro_slope(p0, sA, A, P.q_c, P.a4_c);
  double e0[4], eL[4], eR[4], eb[4], eA[4], qh[2];
  mpsi<false>(mu, mv, 1, 0, xi, e0);
  mpsi_c<false>(mp, mv, 2, 0, xi, aL, eL);
  mpsi_c<false>(mn, mv, 2, 0, xi, aR, eR);
  mpsi_c<false>(mu, mv, 1, 1, xi, b, eb);
  mpsi_c<false>(mu, mv, 1, 0, xi, A, eA);
  face_heat(P, p0, W0, Q1, T3, qh);
  macro_flux(P, p0, Mt, e0, eL, eR, eb, eA, Q1, Q2, qh, len, F);
  fold_record<false>(P, p0, xi, Mt, aL, aR, b, A, qh, len, false, rec);
  U0 = p0.U;
  V0 = p0.V;
}

// One interface of a solver: face (i, j) of the x family (the left face of cell (i, j), i up to
// nx) or of the y family (its lower face, j up to ny), number e of its family.
template <bool kX>
struct Face {
  static constexpr bool x = kX;
  int i, j;
  size_t e, nf;        // number in the family, faces of the family
  bool gl, gr;         // the side below / above is a channel's inlet / outlet ghost column
  bool wall;           // a channel wall
  unsigned cl, cr;     // the cells below and above (periodic images; a ghost's cell of the
                       // moment sums; beyond a wall some cell, unused)
};
template <bool x>
__device__ __forceinline__ Face<x> face_at(const KParams& P, long e) {
  Face<x> f;
  const bool chan = P.bc == UGKS_BC_CHANNEL;
  const int row = x ? P.nx + 1 : P.nx;
  f.e = (size_t)e;
  f.nf = x ? (size_t)P.ny * (P.nx + 1) : (size_t)(P.ny + 1) * P.nx;
  f.j = (int)(e / row);
  f.i = (int)(e - (long)f.j * row);
  f.gl = x && chan && f.i == 0;
  f.gr = x && chan && f.i == P.nx;
  f.wall = !x && chan && (f.j == 0 || f.j == P.ny);
  const unsigned ghost = (unsigned)P.nc + f.j;
  if (x) {
    f.cl = f.gl ? ghost : (unsigned)(f.j * P.nx + wrap(f.i - 1, P.nx));
    f.cr = f.gr ? ghost : (unsigned)(f.j * P.nx + wrap(f.i, P.nx));
  } else {
    f.cl = (unsigned)(wrap(f.j - 1, P.ny) * P.nx + f.i);
    f.cr = (unsigned)(wrap(f.j, P.ny) * P.nx + f.i);
  }
  return f;
}

// W of the cells (or ghosts) below and above a face, in its local frame.
template <bool kX>
__device__ __forceinline__ void face_sides(const Inst* __restrict__ I, const KParams& P,
                                           int parity, const Face<kX>& f, double* wl,
                                           double* wr) {
  const UGKS_GLOBAL double* W = I->W[parity];
  const UGKS_GLOBAL double* Wg = I->Wg;
  const UGKS_GLOBAL double* WL = f.gl ? Wg + 4 * (size_t)f.j : W + 4 * (size_t)f.cl;
  const UGKS_GLOBAL double* WR = f.gr ? Wg + 4 * ((size_t)P.ny + f.j) : W + 4 * (size_t)f.cr;
  const int n = f.x ? 1 : 2, t = 3 - n;
  wl[0] = WL[0];
  wl[1] = WL[n];
  wl[2] = WL[t];
  wl[3] = WL[3];
  wr[0] = WR[0];
  wr[1] = WR[n];
  wr[2] = WR[t];
  wr[3] = WR[3];
}

// Records of one face.  With internal degrees of freedom each face also gets the record of H, nf
// records after that of G; it repeats the macroscopic flux, so either record serves Eq. (4).
template <bool kX>
__device__ __forceinline__ RecRef record_at(const Inst* __restrict__ I, const Face<kX>& f, int c) {
  return RecRef{(kX ? I->recx : I->recy) + f.e + (size_t)c * f.nf * kRec, f.nf};
}
// The macroscopic flux F in the local frame.
template <bool kX>
__device__ __forceinline__ void put_flux(const RecRef& r, const double* F) {
  r[R_FX + 0] = F[0];
  r[kX ? R_FX + 1 : R_FX + 2] = F[1];
  r[kX ? R_FX + 2 : R_FX + 1] = F[2];
  r[R_FX + 3] = F[3];
}
// The interface velocity in the local frame.
template <bool kX>
__device__ __forceinline__ void put_velocity(const RecRef& r, double U0, double V0) {
  r[kX ? R_UX : R_VY] = U0;
  r[kX ? R_VY : R_UX] = V0;
}

// The record(s) of a channel wall from the sums S of its cell.
template <bool kX>
__device__ __forceinline__ void wall_record(const Inst* __restrict__ I, const KParams& P,
                                            double dt, const Face<kX>& f, const double* S) {
  const RecRef rec = record_at(I, f, 0), recH = record_at(I, f, 1);
  // diffuse wall: sums of the wall-row cell towards the wall; local frame (v, u)
  const bool top = f.j == P.ny;
  const double* Q1 = S + 8;
  const double den = top ? P.wall_den_top : P.wall_den_bot;
  const double* Gw = top ? P.wall_G_top : P.wall_G_bot;
  const double rho_w = -Q1[0] / den;
  const double s = P.dx * dt;
  double Fl[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) Fl[q] = s * (Q1[q] + rho_w * Gw[q]);
  // H leaves the wall with kap_w times the Maxwellian of G
  for (int c = 0; c < P.NC; ++c) {
    const RecRef r = c ? recH : rec;
    put_flux<kX>(r, Fl);
    r[R_GC] = s * rho_w * P.lam_w / kPi * (c ? P.kap_w : 1.0);
    r[R_LAM] = P.lam_w;
    r[R_UX] = 0.0;
    r[R_VY] = 0.0;
    r[R_M4] = s;
    r[R_M5] = 0.0;
    r[R_KIND] = K_WALL;
#pragma unroll
    for (int q = 0; q < 13; ++q) r[R_E + q] = 0.0;  // a wall carries no polynomial
  }
  if (!(rho_w > 0.0) || !isfinite(rho_w)) *P.flag = 1;
}

// The record(s) of an interior face of a collisionless gas from its sums S.
template <bool kX>
__device__ __forceinline__ void free_record(const Inst* __restrict__ I, const KParams& P,
                                            double dt, const Face<kX>& f, const double* S) {
  const RecRef rec = record_at(I, f, 0), recH = record_at(I, f, 1);
  double F[4];
  free_flux(dt, S + 8, S + 12, kX ? P.dy : P.dx, P.NC, F, rec, recH);
  for (int c = 0; c < P.NC; ++c) {
    put_flux<kX>(c ? recH : rec, F);
    put_velocity<kX>(c ? recH : rec, 0.0, 0.0);
  }
}

// The record of one face from its sums S (both sides added; a wall: those of its cell) and heat
// sum T3, for solvers with one part of every sum (which have no internal degrees of freedom: H
// makes a second part).
template <bool kX>
__device__ __forceinline__ void face_record(const Inst* __restrict__ I, const KParams& P,
                                            double dt, const Face<kX>& f, const double* S,
                                            double T3, const double* wl, const double* wr) {
  if (f.wall) {
    wall_record(I, P, dt, f, S);
    return;
  }
  if (P.collisionless) {
    free_record(I, P, dt, f, S);
    return;
  }
  const RecRef rec = record_at(I, f, 0);
  double F[4], U0, V0;
  interface_scalars(P, dt, S, wl, wr, kX ? P.dx : P.dy, kX ? P.dy : P.dx, F, rec, U0, V0, T3);
  put_flux<kX>(rec, F);
  put_velocity<kX>(rec, U0, V0);
}

// The update kernel of this step takes the max rate of W^{n+1} into the other slot.
__device__ __forceinline__ void clear_rate(const KParams& P, int parity) {
  P.rmax[parity ^ 1] = 0ull;
}

// Instances with one part of every sum: one thread per interface, the workgroups of the x faces
// (ny rows of nx+1) first, then those of the y faces (ny+1 rows of nx).
template <bool kX>
__device__ __forceinline__ void face_direct(const Inst* __restrict__ I, const KParams& P,
                                            int parity, long e) {
  const Face<kX> f = face_at<kX>(P, e);
  if (e >= (long)f.nf) return;
  // a wall takes the sums of its cell alone, which lies above the bottom and below the top
  const bool nol = f.wall && f.j == 0, nor = f.wall && f.j != 0;
  auto sum = [&](int side, int q, unsigned c) {
    return ldb((const UGKS_GLOBAL double*)I->hs + sum_at<kX>(P, side, q), c * 8u);
  };
  double S[16], T3 = 0.0, wl[4], wr[4];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const double a = sum(kX ? S_XP : S_YP, q, f.cl), c = sum(kX ? S_XM : S_YM, q, f.cr);
    S[q] = nol ? c : (nor ? a : a + c);
  }
  if (P.shak) T3 = sum(kX ? S_XP : S_YP, 16, f.cl) + sum(kX ? S_XM : S_YM, 16, f.cr);
  face_sides(I, P, parity, f, wl, wr);
  face_record(I, P, step_dt(P, parity), f, S, T3, wl, wr);
}
__global__ __launch_bounds__(256) void faces_kernel(const Inst* inst, const int* off,
                                                    int ninst, int step) {
  const int b = blockIdx.x;
  const int ii = find_inst(off, ninst, b);
  const Inst* __restrict__ I = inst + ii;
  const KParams P = I->P;
  const int parity = (I->cur + step) & 1;
  const int local = b - first_block(off, ii);
  if (local == 0 && threadIdx.x == 0) clear_rate(P, parity);
  const int bx = (P.ny * (P.nx + 1) + 255) / 256;
  if (local < bx)
    face_direct<true>(I, P, parity, (long)local * 256 + threadIdx.x);
  else
    face_direct<false>(I, P, parity, (long)(local - bx) * 256 + threadIdx.x);
}

// The chain of interface_scalars for kF faces of one family, with its independent parts on the kNW
// wavefronts of a workgroup (lanes: faces).  The chain is about 2000 FP64 instructions, each issued
// over four clocks: 3.7 us for one wavefront, on one SIMD of a CU whose others have nothing to do.
// In three stages, handed on in LDS, the interface kernel of 40 x 10 cells takes 9.6 us instead of
// 11.1, of 80 x 40 11.2 instead of 13.7.  erfc and the recurrences of the axis moments on one
// wavefront, both in the first stage, made it the longest: 10.2 and 11.7.  Every value is formed by
// the expressions of interface_scalars, and the same in all forms.  With kNW = 4 a wavefront takes
// the parts of two of eight (r).
enum ChainRow {
  X_A = 0,        // aL, aR, b: 4 each
  X_MT = 12,      // Mt: 5
  X_C = 17,       // c[2..6] of the axis moments
  X_M0 = 22,      // mp[0], mn[0]
  X_EDGE = 24,
  X_M = 25,       // m1, m2, m3: 4 each
  X_E = 37,       // eL, eR, eb, e0: 4 each
  X_COUNT = 53
};
template <bool kXi, bool kX, int kF, int kNW>
__device__ __forceinline__ void faces_staged(const Inst* __restrict__ I, const KParams& P,
                                             double dt, const Face<kX>& f, bool writes, int fl,
                                             bool active, int w, const double* wl,
                                             const double* wr, const double (*red)[kF],
                                             double (*ch)[kF]) {
  const double dn = kX ? P.dx : P.dy, len = kX ? P.dy : P.dx;
  const int r = kNW == 8 ? w - 4 : w;  // second part of a stage
  auto sum = [&](int q) { return red[q][fl] + red[16 + q][fl]; };
  double W0[4];
  Prim p0;
  Xi xi;
  // stage 1: micro slopes (wavefronts 0 to 2), time weights, moments along the axes
  if (active) {
#pragma unroll
    for (int q = 0; q < 4; ++q) W0[q] = sum(q);
    const bool ok = prim_of(W0, p0, P.lam_c);
    xi = xi_of<kXi>(P, p0);
    if (w < 3) {
      // aL and aR from the differences to the cells' W, b from the sums' time derivative
      double sw[4], a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double d = w == 0 ? W0[q] - wl[q] : wr[q] - W0[q];
        sw[q] = w == 2 ? sum(4 + q) : d / (0.5 * dn);
      }
      micro_slope(p0, sw, a, P.q_c, P.a4_c);
#pragma unroll
      for (int q = 0; q < 4; ++q) ch[X_A + 4 * w + q][fl] = a[q];
    } else if (w == 3) {
      if (writes && !ok) *P.flag = 1;
      double Mt[5];
      time_weights(dt, collision_time(p0, P.mu_ref), Mt);
#pragma unroll
      for (int q = 0; q < 5; ++q) ch[X_MT + q][fl] = Mt[q];
    }
    if (r == 0 || r == 1) {
      ch[X_M0 + r][fl] = axis_m0(p0.U, p0.lam, r);
    } else if (r == 2) {
      double c[7];
      axis_factors(p0.lam, c);
#pragma unroll
      for (int n = 2; n < 7; ++n) ch[X_C + n - 2][fl] = c[n];
    } else if (r == 3) {
      ch[X_EDGE][fl] = axis_edge(p0.U, p0.lam);
    }
  }
  __syncthreads();
  double c[7], mu[7], mv[7];
  // stage 2: moments of the slopes
  if (active) {
#pragma unroll
    for (int n = 2; n < 7; ++n) c[n] = ch[X_C + n - 2][fl];
    axis_full(p0.U, c, mu);
    axis_full(p0.V, c, mv);
    double o[4];
    if (w == 0 || w == 1 || r == 0 || r == 1) {
      const int k = w == 0 || r == 0 ? 0 : 1;
      double m[7], a[4];
      axis_half_line(p0.U, c, ch[X_M0 + k][fl], ch[X_EDGE][fl], k, m);
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = ch[X_A + 4 * k + q][fl];
      if (w < 2) {
        mpsi_c<kXi>(m, mv, 1, 0, xi, a, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) ch[X_M + 4 * k + q][fl] = o[q];
      }
      if (r >= 0) {
        mpsi_c<kXi>(m, mv, 2, 0, xi, a, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) ch[X_E + 4 * k + q][fl] = o[q];
      }
    } else if (w == 2 || r == 2) {
      double b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = ch[X_A + 8 + q][fl];
      if (w == 2) {
        mpsi_c<kXi>(mu, mv, 0, 1, xi, b, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) ch[X_M + 8 + q][fl] = o[q];
      }
      if (r == 2) {
        mpsi_c<kXi>(mu, mv, 1, 1, xi, b, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) ch[X_E + 8 + q][fl] = o[q];
      }
    } else if (w == 3) {
      mpsi<kXi>(mu, mv, 1, 0, xi, o);
#pragma unroll
      for (int q = 0; q < 4; ++q) ch[X_E + 12 + q][fl] = o[q];
    }
  }
  __syncthreads();
  // stage 3: A, then the macroscopic flux (wavefront 0) and the polynomial of G (1) and H (2)
  if (w > (kXi ? 2 : 1) || !writes) return;
  double sA[4], A[4], Mt[5], Q1[4], qh[2];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    sA[q] = -p0.rho * (ch[X_M + q][fl] + ch[X_M + 4 + q][fl] + ch[X_M + 8 + q][fl]);
  micro_slope(p0, sA, A, P.q_c, P.a4_c);
#pragma unroll
  for (int q = 0; q < 5; ++q) Mt[q] = ch[X_MT + q][fl];
#pragma unroll
  for (int q = 0; q < 4; ++q) Q1[q] = sum(8 + q);
  face_heat(P, p0, W0, Q1, P.shak ? red[32][fl] + red[33][fl] : 0.0, qh);
  if (w == 0) {
    double eA[4], e[4][4], Q2[4], F[4];
    mpsi_c<kXi>(mu, mv, 1, 0, xi, A, eA);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int q = 0; q < 4; ++q) e[k][q] = ch[X_E + 4 * k + q][fl];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) Q2[q] = sum(12 + q);
    macro_flux(P, p0, Mt, e[3], e[0], e[1], e[2], eA, Q1, Q2, qh, len, F);
#pragma unroll
    for (int k = 0; k < (kXi ? 2 : 1); ++k) put_flux<kX>(record_at(I, f, k), F);
  } else {
    double a[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
      for (int q = 0; q < 4; ++q) a[k][q] = ch[X_A + 4 * k + q][fl];
    }
    const RecRef rec = record_at(I, f, w - 1);
    fold_record<kXi>(P, p0, xi, Mt, a[0], a[1], a[2], A, qh, len, w == 2, rec);
    put_velocity<kX>(rec, p0.U, p0.V);
  }
}

// Instances whose moment kernel leaves several parts of every sum (velocity chunks, the chunks of
// H): a workgroup takes kF faces of one family.  Its threads first add the parts of the faces' 32
// sums (16 from each side) in chunk order, kIt sums a thread, all loads of a sum in flight at once;
// they meet in LDS, and the wavefronts go on to the records together (faces_staged).  Each sum is
// towards one face, so no part is read twice and no launch of its own is needed for the sums (it
// took 4.6 us of launch and latency on any mesh).  What is left is bound by latency: 1.2 us for the
// plan, 2 for the sums, 2.5 for faces_staged.  On a small mesh with many parts (40 x 20: 14) 64
// faces a workgroup would have 27 CUs read everything (4.3 us for the sums), so the plan takes 16
// or 32 faces there.  The Shakhov model's cell moments, which the update kernel reads, are added by
// the workgroups after those of the faces, one thread per moment and cell.
template <bool kX, int kF, int kNW>
__device__ __forceinline__ void faces_of_chunks(const Inst* __restrict__ I, const KParams& P,
                                                int parity, long first, int lane, int w,
                                                double (*red)[kF], double (*ch)[kF]) {
  constexpr int kSub = kWave / kF;            // sums a wavefront takes side by side
  constexpr int kStep = kNW * kSub, kIt = 32 / kStep;
  const int n = I->gsplit * P.NC;
  const long nf = kX ? (long)P.ny * (P.nx + 1) : (long)(P.ny + 1) * P.nx;
  const int fl = lane % kF, sub = lane / kF;
  const bool mine = first + fl < nf;
  const Face<kX> f = face_at<kX>(P, mine ? first + fl : nf - 1);
  double wl[4], wr[4];
  if (w < 2) face_sides(I, P, parity, f, wl, wr);
  // Sums u0 + it kStep from `first` on (u < half: sum u of the cell below the face, else sum u - half
  // of the cell above it; those of one face family follow one another, stride values apart) into the
  // rows of `out`, up to kParts parts at a time (past the last part it is read again and not added).
  // With kF = 64 a wavefront's sum is uniform and its place goes into the base; else it is a lane's,
  // in the 32-bit offset (the plan sees to the size).
  const long long stride = kX ? P.nc + P.ny : P.nc;
  auto add = [&](const UGKS_GLOBAL double* first, int half, double (*out)[kF], int u0,
                 auto count_c, auto parts_c) {
    constexpr int kN = decltype(count_c)::value, kParts = decltype(parts_c)::value;
    const UGKS_GLOBAL double* base[kN];
    unsigned off[kN];
    double a[kN];
#pragma unroll
    for (int it = 0; it < kN; ++it) {
      const int u = u0 + it * kStep;
      const unsigned c = u >= half ? f.cr : f.cl;
      base[it] = first + (kSub == 1 ? u * stride : 0);
      off[it] = ((kSub == 1 ? 0u : (unsigned)(u * stride)) + c) * 8u;
      a[it] = 0.0;
    }
    long long at = 0;
    for (int g0 = 0; g0 < n; g0 += kParts) {
      double v[kN][kParts];
#pragma unroll
      for (int k = 0; k < kParts; ++k) {
#pragma unroll
        for (int it = 0; it < kN; ++it) v[it][k] = ldb(base[it] + at, off[it]);
        at += g0 + k + 1 < n ? P.part : 0;
      }
#pragma unroll
      for (int k = 0; k < kParts; ++k) {
#pragma unroll
        for (int it = 0; it < kN; ++it) a[it] += g0 + k < n ? v[it][k] : 0.0;
      }
    }
#pragma unroll
    for (int it = 0; it < kN; ++it) out[u0 + it * kStep][fl] = a[it];
  };
  using It = std::integral_constant<int, kIt>;
  const int u0 = w * kSub + sub;
  const UGKS_GLOBAL double* sums = I->hs + sum_at<kX>(P, kX ? S_XP : S_YP, 0);
  if (n <= 2)
    add(sums, 16, red, u0, It(), std::integral_constant<int, 2>());
  else if (n <= 4)
    add(sums, 16, red, u0, It(), std::integral_constant<int, 4>());
  else if (n <= 6 || kIt == 8)
    add(sums, 16, red, u0, It(), std::integral_constant<int, 6>());
  else if (n <= 9)
    add(sums, 16, red, u0, It(), std::integral_constant<int, 9>());
  else if (n <= 12)
    add(sums, 16, red, u0, It(), std::integral_constant<int, 12>());
  else
    add(sums, 16, red, u0, It(), std::integral_constant<int, 16>());
  if (P.shak && w >= kNW - 2 && sub == 0)  // the heat sums, in rows 32 and 33
    add(I->hs + sum_at<kX>(P, kX ? S_XP : S_YP, 16), 1, red + 32, w - (kNW - 2),
        std::integral_constant<int, 1>(), std::integral_constant<int, 8>());
  __syncthreads();
  const double dt = step_dt(P, parity);
  if (!P.collisionless) {
    if (P.NC > 1)
      faces_staged<true, kX, kF, kNW>(I, P, dt, f, sub == 0 && mine && !f.wall, fl, sub == 0, w,
                                      wl, wr, red, ch);
    else
      faces_staged<false, kX, kF, kNW>(I, P, dt, f, sub == 0 && mine && !f.wall, fl, sub == 0, w,
                                       wl, wr, red, ch);
    if (kX || !f.wall) return;
  }
  if (w != 0 || sub != 0 || !mine) return;
  // a wall takes the sums of its cell alone, which lies above the bottom and below the top
  const bool nol = f.wall && f.j == 0, nor = f.wall && f.j != 0;
  double S[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const double a = red[q][fl], c = red[16 + q][fl];
    S[q] = nol ? c : (nor ? a : a + c);
  }
  if (f.wall)
    wall_record(I, P, dt, f, S);
  else
    free_record(I, P, dt, f, S);
}

template <int kF, int kNW>
__global__ __launch_bounds__(kWave* kNW)
__attribute__((amdgpu_waves_per_eu(2))) void faces_kernel_chunks(const Inst* inst,
                                                                  const int* off, int ninst,
                                                                  int step) {
  __shared__ double red[34][kF];
  __shared__ double ch[X_COUNT][kF];
  const int b = blockIdx.x;
  const int ii = find_inst(off, ninst, b);
  const Inst* __restrict__ I = inst + ii;
  const KParams P = I->P;
  const int parity = (I->cur + step) & 1;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int local = b - first_block(off, ii);
  if (local == 0 && threadIdx.x == 0) clear_rate(P, parity);
  const int bx = (P.ny * (P.nx + 1) + kF - 1) / kF;
  const int by = ((P.ny + 1) * P.nx + kF - 1) / kF;
  if (local < bx) {
    faces_of_chunks<true, kF, kNW>(I, P, parity, (long)local * kF, lane, w, red, ch);
    return;
  }
  if (local < bx + by) {
    faces_of_chunks<false, kF, kNW>(I, P, parity, (long)(local - bx) * kF, lane, w, red,
                                    ch);
    return;
  }
  const int n = I->gsplit * P.NC;
  const long long e = (long long)(local - bx - by) * (kWave * kNW) + threadIdx.x;
  if (e >= (long long)(kSlotsShakhov - kSlotCell) * P.nc) return;
  UGKS_GLOBAL double* at = I->hs + cell_sum_at(P, 0) + e;
  double x = at[0];
  for (int g0 = 1; g0 < n; g0 += 8) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = g0 + k < n ? at[(g0 + k) * P.part] : 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (g0 + k < n) x += v[k];
  }
  at[0] = x;
}

// ------------------------------------------------------------------ update kernel
// A workgroup takes one segment of kTileU cells of two neighbouring rows, jb and jb + 1; its
// lanes hold the segment and two cells on each side.  Wavefront q runs velocity quadrant q
// (signs su, sv) over both rows: u nodes outer, v nodes inner.  The upwind row of the pair
// (jb for sv > 0) comes first: the flux through the face between the two rows is evaluated
// once, as that row's outgoing flux, and taken over in registers as the other row's incoming
// flux.  Per velocity the wavefront loads five row segments of the plane (the pair, the two
// rows upwind of it, the row downwind of it) instead of four per row.
//
// Arithmetic: with f stored in FP64 every step is FP64.  With f stored in FP32 the
// per-velocity work (slopes, reconstruction, face fluxes, Eq. (3)) runs in FP32 on FP32
// copies of the face records and cell constants; Eq. (4), the interface scalars and the
// velocity moments stay FP64.
//
// Rows: the pairs are (0, 1), (2, 3), ...; with ny odd the last pair is (ny - 2, ny - 1), of
// which only row ny - 1 is written (row ny - 2 belongs to the pair before), and with ny = 1
// the only pair is (-1, 0), of which only row 0 is written.  A row outside the mesh reads
// zeros or halo values and writes nothing; the faces it touches are chosen so that no flux
// that a written row takes from it depends on its values (see face_role).
constexpr int kPair = 2;
// Face record fields staged in LDS: R_GC .. R_M5 except R_VY (read once, for the Gauss starts).
constexpr int kSF = R_M5 - R_GC;
__host__ __device__ constexpr int sf(int R) { return R < R_VY ? R - R_GC : R - R_GC - 1; }
// Per-cell state of Eq. (3) (CellField) for the two rows.
enum CellField { C_LAMN, C_UN, C_VN, C_LAM1, C_U1, C_V1, C_AN, C_A1, C_AF, C_ADF, C_COUNT };
template <typename T>
struct PairStage {
  T sx[kPair][kSF][kWave + 1];  // x face i0 - 2 + f of row jb + r (left face of lane f)
  T sy[kPair + 1][kSF][kWave];  // y face row jb + r (bottom face of row jb + r), lane l
  T cell[kPair][C_COUNT][kWave];
  // Gauss starts (value, ratio) at the first node of v half h (0: v > 0, 1: v < 0)
  T xs[2][kPair][2][kWave + 1];   // x faces
  T ys[2][kPair + 1][2][kWave];   // y faces
  T gs[2][kPair][2][2][kWave];    // g^n (0) and g^{n+1} (1) of each cell
  // the Gauss recurrences' second factors, exp(-2 lam h^2) - 1: the same in both halves of v
  // and at every u node, so formed once per workgroup and not by every wavefront
  T qx[kPair][kWave + 1];
  T qy[kPair + 1][kWave];
};
// Those of each cell's g^n (0) and g^{n+1} (1), the last of the stage.
template <typename T>
using CellFactors = T[2][kWave];

// A Gaussian factor exp(-lam (x - c)^2) along the uniform nodes x0, x0 + h, x0 + 2h, ...:
// e is its value at the current node and r the ratio to the next one; successive ratios
// differ by the factor exp(-2 lam h^2), applied as r + r (exp(-2 lam h^2) - 1) with the
// second factor from expm1, so that it adds one rounding per node and no drift.
template <typename T>
__device__ __forceinline__ void gauss_next(T& e, T& r, T qm1) {
  e *= r;
  r = fma(r, qm1, r);
}

// The second factor, exp(-2 lam h^2) - 1, in the arithmetic type.
template <typename T>
__device__ __forceinline__ T second_factor(double hstep, double lam) {
  const T h = T(hstep);
  return expm1_of(T(-2) * h * h * T(lam));
}

// Cubic of the folded equilibrium polynomial P(un, ut) of a record (interface scalars) in
// one velocity with the other fixed.  The e1, e4, e5, e7 of the side the particles come from
// are passed in (pos: un > 0).
template <typename T>
struct Cubic {
  T c0, c1, c2, c3;
};
// P as a cubic in the tangential velocity at fixed normal velocity un.
template <typename T>
__device__ __forceinline__ Cubic<T> cubic_in_ut(const T* e, T un) {
  const T h = T(0.5);
  Cubic<T> c;
  c.c0 = fma(un, fma(un, fma(un, h * e[7], e[4] + h * e[3]), e[1]), e[0]);
  c.c1 = fma(un, fma(un, h * e[8], e[5]), e[2]);
  c.c2 = fma(un, h * e[7], e[6] + h * e[3]);
  c.c3 = h * e[8];
  return c;
}
// P as a cubic in the normal velocity at fixed tangential velocity ut.
template <typename T>
__device__ __forceinline__ Cubic<T> cubic_in_un(const T* e, T ut) {
  const T h = T(0.5);
  Cubic<T> c;
  c.c0 = fma(ut, fma(ut, fma(ut, h * e[8], h * e[3] + e[6]), e[2]), e[0]);
  c.c1 = fma(ut, fma(ut, h * e[7], e[5]), e[1]);
  c.c2 = fma(ut, h * e[8], h * e[3] + e[4]);
  c.c3 = h * e[7];
  return c;
}
template <typename T>
__device__ __forceinline__ T horner(const Cubic<T>& c, T x) {
  return fma(x, fma(x, fma(x, c.c3, c.c2), c.c1), c.c0);
}
template <typename T>
__device__ __forceinline__ Cubic<T> scaled(Cubic<T> c, T s) {
  c.c0 *= s;
  c.c1 *= s;
  c.c2 *= s;
  c.c3 *= s;
  return c;
}
// e0..e8 of a staged record for particles with normal velocity of sign s
template <typename T, int N>
__device__ __forceinline__ void load_e(const T (*st)[N], int col, int s, T* e) {
#pragma unroll
  for (int n = 0; n < 9; ++n) e[n] = st[sf(R_E + n)][col];
  if (s < 0) {
    e[1] = st[sf(R_ER + 0)][col];
    e[4] = st[sf(R_ER + 1)][col];
    e[5] = st[sf(R_ER + 2)][col];
    e[7] = st[sf(R_ER + 3)][col];
  }
}

// Shakhov: S of one cell at fixed u as a cubic in v.  kqx, kqy = (1 - Pr)(lambda^2/rho) q;
// S = (A + B v)(a2 v^2 + a1 v + a0) with A + B v = k (c . q), a2 v^2 + a1 v + a0 = 2 lambda |c|^2 - 4.
template <typename T>
__device__ __forceinline__ Cubic<T> shakhov_in_v(T u, T kqx, T kqy, T lam, T U, T V) {
  const T du = u - U;
  const T A = fma(du, kqx, -V * kqy), B = kqy;
  const T a2 = T(2) * lam, a1 = T(-4) * lam * V;
  const T a0 = fma(T(2) * lam, fma(du, du, V * V), T(-4));
  Cubic<T> c;
  c.c0 = A * a0;
  c.c1 = fma(A, a1, B * a0);
  c.c2 = fma(A, a2, B * a1);
  c.c3 = B * a2;
  return c;
}

// Role of y face F (between rows F - 1 and F) for particles moving with the sign sv of v.  A
// channel wall emits its Maxwellian when the particles leave it (F = 0 with sv > 0, F = ny with
// sv < 0): the flux is GC Et(u) E(v) alone, with no polynomial and no free transport, and takes
// nothing from the row beyond the wall.  A wall the particles reach (the other two cases)
// takes the first-order free transport of the wall row (its record has no polynomial and M5 = 0;
// the wall row has no y slope).  Every other face is an interior face.
enum FaceRole { F_INTERIOR = 0, F_EMIT = 1, F_ABSORB = 2 };
__device__ __forceinline__ int face_role(const KParams& P, int F, int sv) {
  if (P.bc != UGKS_BC_CHANNEL) return F_INTERIOR;
  if ((F == 0 && sv > 0) || (F == P.ny && sv < 0)) return F_EMIT;
  if ((F == P.ny && sv > 0) || (F == 0 && sv < 0)) return F_ABSORB;
  return F_INTERIOR;
}

// The equilibrium part of a y face at tangential velocity u as a cubic in v, and its free
// transport weights, for particles of v sign sv, by the face's role.
template <typename T>
__device__ __forceinline__ void y_face(const PairStage<T>& st, int fr, int lane, int sv, int role,
                                       T u, Cubic<T>& c, T& m4, T& m5) {
  const T(*r)[kWave] = st.sy[fr];
  const T d = u - r[sf(R_UX)][lane];
  const T Et = r[sf(R_GC)][lane] * exp_of(-r[sf(R_LAM)][lane] * d * d);
  if (role == F_EMIT) {
    c = Cubic<T>{Et, T(0), T(0), T(0)};
    m4 = m5 = T(0);
    return;
  }
  m4 = r[sf(R_M4)][lane];
  if (role == F_ABSORB) {
    c = Cubic<T>{T(0), T(0), T(0), T(0)};
    m5 = T(0);
    return;
  }
  T e[9];
  load_e(r, lane, sv, e);
  c = scaled(cubic_in_un(e, u), Et);
  m5 = r[sf(R_M5)][lane];
}

// Per velocity quadrant (SU = sign of u, sv = sign of v) of a row pair: Eq. (3) for every
// velocity of the quadrant's chunk of u nodes, in the arithmetic type S of the storage.  Per
// velocity and row a lane (cell i) forms
//   its upwind reconstruction and slope term at its outgoing x and y faces,
//   the flux through its outgoing x face, which the downwind lane takes over as its incoming
//   x flux (x faces of the segment are each evaluated once),
//   the flux through its outgoing y face; the upwind row's is the other row's incoming flux,
//   and the upwind row's incoming flux comes from the reconstruction of the cell below it
//   (i, jb - 1) for sv > 0 (above, (i, jb + 2), for sv < 0).
// The equilibrium part of a face flux is GC En(un) Et(ut) P(un, ut): the Gaussian and cubic
// of the u node are formed once per node, those of the v node follow the node by Gauss
// recurrences.
// kAhead: nodes whose loads are in flight ahead of the node computed.  On the
// 400 x 100 x 40^2 channel 2 measured fastest in both storage types (3 ahead: FP64 1% slower,
// FP32 storage 4% slower, its registers then spill); the Shakhov variant has no registers to
// spare beyond 1.  The ring only works because nothing else in the loop is a vector load: the
// next v node is a scalar load (UGKS_CONST), so waiting for it never waits for f loads.
template <typename S, int SU, bool kShak, bool kNode, bool kOwnQ, int kAhead = kShak ? 1 : 2>
__device__ __forceinline__ void pair_quadrant(const KParams& P, const PairStage<S>& st,
                                              const CellFactors<S>* qg,
                                              const S (*sk)[4][kWave], int lane, int sv,
                                              int jb, bool store0, int g, int G, int gv, int Gv,
                                              bool writes, bool ghost_lane, bool late,
                                              const UGKS_GLOBAL S* fin, UGKS_GLOBAL S* fout,
                                              int i) {
  typedef S T;  // arithmetic type of the per-velocity work
  const bool chan = P.bc == UGKS_BC_CHANNEL;
  const int r0 = sv > 0 ? 0 : 1, r1 = 1 - r0;     // rows of the pair, upwind first
  const int j0 = jb + r0, j1 = jb + r1;           // their mesh rows
  const int jB = j0 - sv;                         // the cell upwind of row j0
  // y face rows of the stage: incoming face of j0, the face between the rows, outgoing of j1
  const int fin_r = sv > 0 ? 0 : 2, fout_r = 2 - fin_r, fmid_r = 1;
  const int role_in = face_role(P, jb + fin_r, sv);
  const int role_mid = face_role(P, jb + fmid_r, sv);
  const int role_out = face_role(P, jb + fout_r, sv);
  auto no_wall = [&](int j) { return !(chan && (j == 0 || j == P.ny - 1)); };
  const bool gm = !ghost_lane;  // ghost columns have zero slopes
  const bool mB = no_wall(jB), m0 = gm && no_wall(j0), m1 = gm && no_wall(j1);
  // cells, and a channel's ghost columns (the ghost Maxwellian of the next step)
  const bool st0 = writes && (r0 == 0 ? store0 : true);
  const bool st1 = writes && (r1 == 0 ? store0 : true);
  // byte offsets of the five rows j0 - 2 sv, j0 - sv, j0, j1 = j0 + sv, j1 + sv
  const unsigned bs = (unsigned)sizeof(S);
  const int ic = plane_col(P, i);
  const int o0 = pidx(P, ic, j0);
  const int L = sv * P.Lx;
  const unsigned oA = (unsigned)(o0 - 2 * L) * bs, oB = (unsigned)(o0 - L) * bs;
  const unsigned oC = (unsigned)o0 * bs, oD = (unsigned)(o0 + L) * bs;
  const unsigned oE = (unsigned)(o0 + 2 * L) * bs;
  const unsigned w0 = st0 ? oC : kDropOffset, w1 = st1 ? oD : kDropOffset;
  const int xo = lane + (SU > 0 ? 1 : 0);  // staged x face the lane's particles leave by
  const T Af0 = st.cell[r0][C_AF][lane], AdF0 = st.cell[r0][C_ADF][lane];
  const T Af1 = st.cell[r1][C_AF][lane], AdF1 = st.cell[r1][C_ADF][lane];
  const Half hu = axis_half(P.K, SU, false), hv = axis_half(P.M, sv, false);
  const int hf = sv > 0 ? 0 : 1;
  const T qx0 = st.qx[r0][xo], qx1 = st.qx[r1][xo];
  const T qyi = st.qy[fin_r][lane], qym = st.qy[fmid_r][lane], qyo = st.qy[fout_r][lane];
  auto cell_factor = [&](int r, int n) {
    if constexpr (kOwnQ)
      return second_factor<T>(P.dv, st.cell[r][n == 0 ? C_LAMN : C_LAM1][lane]);
    else
      return qg[r][n][lane];
  };
  const T qn0 = cell_factor(r0, 0), q10 = cell_factor(r0, 1);
  const T qn1 = cell_factor(r1, 0), q11 = cell_factor(r1, 1);
  const T two_idx = T(2.0 * P.inv_dx), two_idy = T(2.0 * P.inv_dy);
  // this workgroup's v nodes of the half: chunk gv of Gv, vh nodes from node vf
  int vc0, vc1;
  chunk_range(hv.count, gv, Gv, vc0, vc1);
  const int vh = vc1 - vc0, vf = hv.first + vc0 * hv.step;
  // Chunk g of the quadrant: whole u lines, or (kNode, chosen by the plan where the lines do
  // not divide evenly) its share of all nodes, which may start and end inside a line, at the
  // groups of NB nodes that the loop below takes at a time: every node is then computed at the
  // same place of the unrolled loop, with the same rounding, however the chunks lie.
  constexpr int NB = kAhead + 1;
  const int vg = (vh + NB - 1) / NB;  // groups of a line
  int a, vs = 0, left;  // the first line, its first group, groups to compute
  if constexpr (kNode) {
    int n0, n1;
    chunk_range(hu.count * vg, g, G, n0, n1);
    a = n0 / vg;
    vs = n0 - a * vg;
    left = n1 - n0;
  } else {
    int a1;
    chunk_range(hu.count, g, G, a, a1);
    left = (a1 - a) * vg;
  }
  // The two wavefronts of a SIMD are issued oldest first, so the later one falls behind and
  // works on alone, without a partner to fill its waits, once the other has ended.  It goes first
  // over the first half of its chunk, and both end at about the same time: update of 130 x 37
  // cells at 40^2 (Shakhov) 59.0 -> 54.9 us, 96 x 80 periodic at 33^2 52.3 -> 49.4, 200 x 50 at
  // 101^2 544 -> 535, 400 x 100 at 40^2 327 -> 323 (FP64).
  const int lead_to = left - left / 2;
  for (; left > 0; ++a) {
    if (late) {
      if (left > lead_to)
        __builtin_amdgcn_s_setprio(1);
      else
        __builtin_amdgcn_s_setprio(0);
    }
    const int k = hu.first + a * hu.step;
    const int c0 = vs * NB, vn = min(vh - c0, left * NB);  // vn nodes of this line, from node c0
    const int v0 = vf + c0 * hv.step;
    const T u = T(((const UGKS_CONST double*)P.uk)[k]);  // a scalar load
    const T au = fabs(u);
    const T ucx = u * two_idx;
    struct Vals {
      S A, B, C, D, E;  // rows j0 - 2 sv, j0 - sv, j0, j1, j1 + sv
    };
    // planes (read and written) and v nodes are walked with running pointers
    const long long pstep = (long long)hv.step * P.PS;
    const UGKS_GLOBAL S* pnext = plane_of(fin, P, k * P.M + v0);
    UGKS_GLOBAL S* wcur = plane_of(fout, P, k * P.M + v0);
    const UGKS_CONST double* vp = (const UGKS_CONST double*)(P.vm + v0);
    // loads run kAhead nodes ahead of the node computed; past the last node of the chunk they
    // read its plane again
    int nl = 0;
    auto load_next = [&]() {
      const __amdgpu_buffer_rsrc_t r = plane_rsrc(pnext, P);
      const Vals v{bload_raw(r, oA, S{}), bload_raw(r, oB, S{}), bload_raw(r, oC, S{}),
                   bload_raw(r, oD, S{}), bload_raw(r, oE, S{})};
      if (++nl < vn) pnext += pstep;
      return v;
    };
    // the first nodes' stencil values, requested before the node's tables are formed
    Vals ring[NB];
#pragma unroll
    for (int d = 0; d < kAhead; ++d) ring[d] = load_next();
    // x faces of both rows: cubic in v times GC En(u), with |u| folded in
    Cubic<T> cx0, cx1;
    T m4x0, m5x0, m4x1, m5x1;
    {
      T e[9];
      const T(*x0)[kWave + 1] = st.sx[r0];
      load_e(x0, xo, SU, e);
      const T d = u - x0[sf(R_UX)][xo];
      cx0 = scaled(cubic_in_ut(e, u), x0[sf(R_GC)][xo] * exp_of(-x0[sf(R_LAM)][xo] * d * d) * au);
      m4x0 = x0[sf(R_M4)][xo] * au;
      m5x0 = x0[sf(R_M5)][xo] * au;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      T e[9];
      const T(*x1)[kWave + 1] = st.sx[r1];
      load_e(x1, xo, SU, e);
      const T d = u - x1[sf(R_UX)][xo];
      cx1 = scaled(cubic_in_ut(e, u), x1[sf(R_GC)][xo] * exp_of(-x1[sf(R_LAM)][xo] * d * d) * au);
      m4x1 = x1[sf(R_M4)][xo] * au;
      m5x1 = x1[sf(R_M5)][xo] * au;
    }
    __builtin_amdgcn_sched_barrier(0);
    // y faces: cubic in v at tangential u, times GC Et(u)
    Cubic<T> ci, cm, co;
    T m4i, m5i, m4m, m5m, m4o, m5o;
    y_face(st, fin_r, lane, sv, role_in, u, ci, m4i, m5i);
    __builtin_amdgcn_sched_barrier(0);
    y_face(st, fmid_r, lane, sv, role_mid, u, cm, m4m, m5m);
    __builtin_amdgcn_sched_barrier(0);
    y_face(st, fout_r, lane, sv, role_out, u, co, m4o, m5o);
    __builtin_amdgcn_sched_barrier(0);
    // g^n and g^{n+1} of both cells: u factors (with the Eq. (3) weights) times the v
    // Gaussians' start values
    T en0, rn0, e10, r10, en1, rn1, e11, r11;
    {
      const T(*c0)[kWave] = st.cell[r0];
      const T dn = u - c0[C_UN][lane], d1 = u - c0[C_U1][lane];
      en0 = c0[C_AN][lane] * exp_of(-c0[C_LAMN][lane] * dn * dn) * st.gs[hf][r0][0][0][lane];
      e10 = c0[C_A1][lane] * exp_of(-c0[C_LAM1][lane] * d1 * d1) * st.gs[hf][r0][1][0][lane];
      rn0 = st.gs[hf][r0][0][1][lane];
      r10 = st.gs[hf][r0][1][1][lane];
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      const T(*c1)[kWave] = st.cell[r1];
      const T dn = u - c1[C_UN][lane], d1 = u - c1[C_U1][lane];
      en1 = c1[C_AN][lane] * exp_of(-c1[C_LAMN][lane] * dn * dn) * st.gs[hf][r1][0][0][lane];
      e11 = c1[C_A1][lane] * exp_of(-c1[C_LAM1][lane] * d1 * d1) * st.gs[hf][r1][1][0][lane];
      rn1 = st.gs[hf][r1][0][1][lane];
      r11 = st.gs[hf][r1][1][1][lane];
    }
    // Shakhov: the factors (1 + S) of g^n and g^{n+1} of both cells as cubics in v
    Cubic<T> sn0{}, s10{}, sn1{}, s11{};
    if constexpr (kShak) {
      const T(*c0)[kWave] = st.cell[r0];
      const T(*c1)[kWave] = st.cell[r1];
      sn0 = shakhov_in_v(u, sk[r0][0][lane], sk[r0][1][lane], c0[C_LAMN][lane], c0[C_UN][lane],
                         c0[C_VN][lane]);
      s10 = shakhov_in_v(u, sk[r0][2][lane], sk[r0][3][lane], c0[C_LAM1][lane], c0[C_U1][lane],
                         c0[C_V1][lane]);
      sn1 = shakhov_in_v(u, sk[r1][0][lane], sk[r1][1][lane], c1[C_LAMN][lane], c1[C_UN][lane],
                         c1[C_VN][lane]);
      s11 = shakhov_in_v(u, sk[r1][2][lane], sk[r1][3][lane], c1[C_LAM1][lane], c1[C_U1][lane],
                         c1[C_V1][lane]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // v-direction Gaussians of the faces at the first node of the chunk, and their ratios
    T ex0 = st.xs[hf][r0][0][xo], rx0 = st.xs[hf][r0][1][xo];
    T ex1 = st.xs[hf][r1][0][xo], rx1 = st.xs[hf][r1][1][xo];
    T ei = st.ys[hf][fin_r][0][lane], ri = st.ys[hf][fin_r][1][lane];
    T em = st.ys[hf][fmid_r][0][lane], rm = st.ys[hf][fmid_r][1][lane];
    T eo = st.ys[hf][fout_r][0][lane], ro = st.ys[hf][fout_r][1][lane];
    T vv = T(*vp);
    auto advance = [&]() {
      gauss_next(ex0, rx0, qx0);
      gauss_next(ex1, rx1, qx1);
      gauss_next(ei, ri, qyi);
      gauss_next(em, rm, qym);
      gauss_next(eo, ro, qyo);
      gauss_next(en0, rn0, qn0);
      gauss_next(e10, r10, q10);
      gauss_next(en1, rn1, qn1);
      gauss_next(e11, r11, q11);
    };
    // a chunk that starts inside the line runs its recurrences from the stage's starts, so
    // that the values do not depend on where the chunks end
    if constexpr (kNode)
      for (int n = 0; n < c0; ++n) advance();
    // g^n + g^{n+1} of both cells with one product fused, formed where the recurrences advance
    // to a place of the unrolled loop other than its first
    T gf0{}, gf1{};
    // place: of the node in the unrolled loop, or -1 in its remainder
    auto node = [&](const Vals& x, auto place_c) {
      constexpr int place = decltype(place_c)::value;
      const T vnext = T(vp[hv.step]);  // the next node (read one ahead; past the end a pad)
      const T av = fabs(vv);
      const T avcy = av * two_idy;
      // upwind neighbour of row j0: half-cell changes towards the pair (y) and in x
      const T fBw = from_lower(x.B), fBe = from_upper(x.B);
      const T HxB = half_limited(fBe - x.B, x.B - fBw);
      const T HyB = half_limited(x.C - x.B, x.B - x.A, mB);
      const T DB = fma(ucx, HxB, avcy * HyB);
      const T fhB = x.B + HyB;
      // row j0
      const T fCw = from_lower(x.C), fCe = from_upper(x.C);
      const T HxC = half_limited(fCe - x.C, x.C - fCw, gm);
      const T HyC = half_limited(x.D - x.C, x.C - x.B, m0);
      const T DC = fma(ucx, HxC, avcy * HyC);
      const T fxC = SU > 0 ? x.C + HxC : x.C - HxC;
      const T fhC = x.C + HyC;
      // row j1
      const T fDw = from_lower(x.D), fDe = from_upper(x.D);
      const T HxD = half_limited(fDe - x.D, x.D - fDw, gm);
      const T HyD = half_limited(x.E - x.D, x.D - x.C, m1);
      const T DD = fma(ucx, HxD, avcy * HyD);
      const T fxD = SU > 0 ? x.D + HxD : x.D - HxD;
      const T fhD = x.D + HyD;
      // x faces: outgoing of this lane, incoming from the upwind lane
      const T Fxo0 = fma(ex0, horner(cx0, vv), fma(m4x0, fxC, -m5x0 * DC));
      const T Fxo1 = fma(ex1, horner(cx1, vv), fma(m4x1, fxD, -m5x1 * DD));
      const T Fxi0 = SU > 0 ? from_lower(Fxo0) : from_upper(Fxo0);
      const T Fxi1 = SU > 0 ? from_lower(Fxo1) : from_upper(Fxo1);
      // y faces: into row j0, between the rows, out of row j1
      const T Fyi = av * fma(ei, horner(ci, vv), fma(m4i, fhB, -m5i * DB));
      const T Fym = av * fma(em, horner(cm, vv), fma(m4m, fhC, -m5m * DC));
      const T Fyo = av * fma(eo, horner(co, vv), fma(m4o, fhD, -m5o * DD));
      T g0, g1;
      if constexpr (kShak) {
        g0 = fma(e10, T(1) + horner(s10, vv), en0 * (T(1) + horner(sn0, vv)));
        g1 = fma(e11, T(1) + horner(s11, vv), en1 * (T(1) + horner(sn1, vv)));
      } else {
        g0 = place > 0 ? gf0 : e10 + en0;
        g1 = place > 0 ? gf1 : e11 + en1;
      }
      const T f0 = fma(Af0, x.C, fma(AdF0, (Fxi0 - Fxo0) + (Fyi - Fym), g0));
      const T f1 = fma(Af1, x.D, fma(AdF1, (Fxi1 - Fxo1) + (Fym - Fyo), g1));
      // lanes and rows without a cell to write store past the plane's range (dropped)
      const __amdgpu_buffer_rsrc_t wr = plane_rsrc(wcur, P);
      bstore(wr, w0, f0, S{});
      bstore(wr, w1, f1, S{});
      wcur += pstep;
      vp += hv.step;
      vv = vnext;
      const T pe0 = e10, pr0 = r10, pe1 = e11, pr1 = r11;
      const T pn0 = en0, qr0 = rn0, pn1 = en1, qr1 = rn1;
      advance();
      if constexpr (!kShak && place == 0) {
        gf0 = fma(pe0, pr0, en0);
        gf1 = fma(pe1, pr1, en1);
      } else if constexpr (!kShak && place > 0 && place + 1 < NB) {
        gf0 = fma(pn0, qr0, e10);
        gf1 = fma(pn1, qr1, e11);
      }
    };
    // NB value sets in a ring: slot s holds node c + s, loaded kAhead nodes earlier
    int c = 0;
    for (; c + NB <= vn; c += NB) {
      ring[kAhead] = load_next();
      node(ring[0], std::integral_constant<int, 0>());
      ring[0] = load_next();
      node(ring[1], std::integral_constant<int, 1>());
      if constexpr (NB == 3) {
        ring[1] = load_next();
        node(ring[2], std::integral_constant<int, 2>());
      }
    }
#pragma unroll
    for (int s = 0; s < NB; ++s) {
      if (c + s < vn) {
        ring[(s + kAhead) % NB] = load_next();
        node(ring[s], std::integral_constant<int, -1>());
      }
    }
    left -= vg - vs;
    vs = 0;
  }
}

// Fill mode of the update kernel, quadrant wavefront: the ghost columns of the current f from
// the ghost states of the current W (after the initial state and after a state is set).  It
// forms the ghost lanes' g^{n+1} with the expressions and Gauss recurrences of the update loop,
// where Eq. (3) with every other weight zero leaves f = g^{n+1}, so a state set from a
// checkpoint steps on exactly as a running solver does.
template <typename S, int SU>
__device__ __forceinline__ void ghost_fill_quadrant(const KParams& P, const PairStage<S>& st,
                                                    const CellFactors<S>* qg, int lane, int sv,
                                                    int jb, bool store0, int g, int G, int gv,
                                                    int Gv, bool ghost_w, UGKS_GLOBAL S* f, int i) {
  typedef S T;
  const int r0 = sv > 0 ? 0 : 1, r1 = 1 - r0;
  const int j0 = jb + r0;
  const bool st0 = ghost_w && (r0 == 0 ? store0 : true);
  const bool st1 = ghost_w && (r1 == 0 ? store0 : true);
  const unsigned bs = (unsigned)sizeof(S);
  const int ic = plane_col(P, i);
  const int o0 = pidx(P, ic, j0);
  const unsigned oC = (unsigned)o0 * bs, oD = (unsigned)(o0 + sv * P.Lx) * bs;
  const unsigned w0 = st0 ? oC : kDropOffset, w1 = st1 ? oD : kDropOffset;
  const Half hu = axis_half(P.K, SU, false), hv = axis_half(P.M, sv, false);
  const int hf = sv > 0 ? 0 : 1;
  const T qn0 = qg[r0][0][lane], q10 = qg[r0][1][lane];
  const T qn1 = qg[r1][0][lane], q11 = qg[r1][1][lane];
  const long long pstep = (long long)hv.step * P.PS;
  int a0, a1;
  chunk_range(hu.count, g, G, a0, a1);
  int c0, c1;
  chunk_range(hv.count, gv, Gv, c0, c1);
  const int vn = c1 - c0, vf = hv.first + c0 * hv.step;
  for (int a = a0; a < a1; ++a) {
    const int k = hu.first + a * hu.step;
    const T u = T(((const UGKS_CONST double*)P.uk)[k]);  // a scalar load
    UGKS_GLOBAL S* wcur = plane_of(f, P, k * P.M) + (long long)vf * P.PS;
    T en0, rn0, e10, r10, en1, rn1, e11, r11;
    {
      const T(*c0)[kWave] = st.cell[r0];
      const T dn = u - c0[C_UN][lane], d1 = u - c0[C_U1][lane];
      en0 = c0[C_AN][lane] * exp_of(-c0[C_LAMN][lane] * dn * dn) * st.gs[hf][r0][0][0][lane];
      e10 = c0[C_A1][lane] * exp_of(-c0[C_LAM1][lane] * d1 * d1) * st.gs[hf][r0][1][0][lane];
      rn0 = st.gs[hf][r0][0][1][lane];
      r10 = st.gs[hf][r0][1][1][lane];
    }
    {
      const T(*c1)[kWave] = st.cell[r1];
      const T dn = u - c1[C_UN][lane], d1 = u - c1[C_U1][lane];
      en1 = c1[C_AN][lane] * exp_of(-c1[C_LAMN][lane] * dn * dn) * st.gs[hf][r1][0][0][lane];
      e11 = c1[C_A1][lane] * exp_of(-c1[C_LAM1][lane] * d1 * d1) * st.gs[hf][r1][1][0][lane];
      rn1 = st.gs[hf][r1][0][1][lane];
      r11 = st.gs[hf][r1][1][1][lane];
    }
    for (int c = 0; c < vn; ++c) {
      const T g0 = e10 + en0, g1 = e11 + en1;
      const __amdgpu_buffer_rsrc_t wr = plane_rsrc(wcur, P);
      bstore(wr, w0, g0, S{});
      bstore(wr, w1, g1, S{});
      wcur += pstep;
      gauss_next(en0, rn0, qn0);
      gauss_next(e10, r10, q10);
      gauss_next(en1, rn1, qn1);
      gauss_next(e11, r11, q11);
    }
  }
}

// The body of the update kernel; kShak: the Shakhov collision model; kNode: chunks by node.
template <typename S, bool kShak, int kCh, bool kFill = false, bool kNode = false>
__device__ __forceinline__ void update_body(const Inst* inst, const int* off, int ninst, int step) {
  typedef S T;  // arithmetic type of the per-velocity work (and of the LDS stage)
  __shared__ PairStage<T> st;
  // Shakhov: (1 - Pr)(lambda^2/rho) q of each lane's cell at t^n and t^{n+1}, per row
  __shared__ T sk_raw[kShak ? kPair * 4 * kWave : 1];
  T(*sk)[4][kWave] = reinterpret_cast<T(*)[4][kWave]>(sk_raw);
  // The FP64 Shakhov form of four wavefronts forms the cells' second factors in every wavefront
  // instead: with them in LDS a CU holds one of its workgroups and not two (update of 100 x 60 cells
  // at 11 x 24, 300 workgroups: 48.2 us with them there, 36.5 without; of 40 x 10 at 24^2, 120
  // workgroups: 15.8 and 16.9).
  constexpr bool kOwnQ = sizeof(S) == 8 && kShak && kCh == 1;
  __shared__ T qg_raw[kOwnQ ? 1 : kPair * 2 * kWave];
  CellFactors<T>* qg = reinterpret_cast<CellFactors<T>*>(qg_raw);
  const int lane = threadIdx.x & (kWave - 1);
  // wavefront w: quadrant q, and c, which of the workgroup's kCh velocity chunks
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q = w & 3, c = w >> 2;
  const int ii = find_inst(off, ninst, blockIdx.x);
  const Inst* __restrict__ I = inst + ii;
  const KParams P = I->P;
  const int parity = (I->cur + step) & 1;
  const int G = I->usplit, Gv = P.vsplit;
  const int ntx = (P.nx + kTileU - 1) / kTileU;
  const int b = xcd_block(blockIdx.x - first_block(off, ii),
                          ntx * ((P.ny + 1) / 2) * G * Gv * P.NC);
  int t, gg, pb;
  cell_block(b, (P.ny + 1) / 2, ntx, t, gg, pb);
  const int jb = min(2 * pb, P.ny - 2);       // rows jb, jb + 1
  const bool store0 = jb == 2 * pb && jb >= 0;  // row jb is this pair's to write
  // chunk gg: u chunk g of G fastest, then v chunk gv of Gv; chunks G Gv.. update H: its
  // planes, its face records, its equilibria
  const bool hpart = gg >= G * Gv;
  const int g2 = hpart ? gg - G * Gv : gg;
  const int g = g2 % G, gv = g2 / G;
  const long long hoff = hpart ? (long long)P.NV * P.PS : 0ll;
  const UGKS_GLOBAL S* fin = static_cast<const UGKS_GLOBAL S*>(I->f[parity]) + hoff;
  // fill mode writes the ghost columns of the current f
  UGKS_GLOBAL S* fout = static_cast<UGKS_GLOBAL S*>(I->f[kFill ? parity : parity ^ 1]) + hoff;
  // face records, field-major (RecRef): field f of x face e at f nfx + e, of y face e at
  // f nfy + e; the records of H follow those of G
  const size_t nfx = (size_t)P.ny * (P.nx + 1), nfy = (size_t)(P.ny + 1) * P.nx;
  const UGKS_GLOBAL double* recx = I->recx + (hpart ? nfx * kRec : (size_t)0);
  const UGKS_GLOBAL double* recy = I->recy + (hpart ? nfy * kRec : (size_t)0);
  const UGKS_GLOBAL double* W = I->W[parity];
  UGKS_GLOBAL double* Wout = I->W[parity ^ 1];
  const int i0 = t * kTileU;
  const int i = i0 - kHalo + lane;
  const bool valid = lane >= kHalo && lane < kHalo + kTileU && i < P.nx;
  const bool chan = P.bc == UGKS_BC_CHANNEL;
  const bool ghost_lane = chan && (i == -1 || i == P.nx);
  // the ghost lane whose neighbouring cell is this segment's writes the ghost column (the
  // outlet column can also be the right halo of the segment before the last)
  const bool ghost_w = ghost_lane && (i < 0 || lane <= kHalo + kTileU);
  // The prologue fills the stage with one barrier at its end.  Its parts do not read one another's
  // LDS, so each wavefront first requests the inputs of its own part, then its share of the
  // face records, works while those are in flight, and writes them to LDS last.  Parts:
  //   wavefronts 0, 1   Eq. (4) and the cells' data of row jb + w, the Gauss starts of g^{n+1}
  //   face units        the Gauss starts of 64 faces: x faces of row jb + r (unit r) and y face
  //                     row jb + r (unit 2 + r); with eight wavefronts one unit to each of 2..6,
  //                     with four 2 1/2 units (a half: one half of v) to each of 2, 3
  //   g^n starts        wavefront 7, or with four wavefronts with the cells of each row
  // What bounds it is the longest chain of dependent FP64 work (Eq. (4), two states, eight
  // exponentials) on otherwise idle SIMDs; with the g^n starts and the recurrence factors (nine
  // expm1 that every wavefront formed for itself) shared out, the update of 40 x 20 cells at
  // 29^2 went from 22.3 to 20.3 us, of 400 x 100 at 40^2 from 332 to 327 us (FP64).
  double eWn[kPair][4] = {{1.0, 0.0, 0.0, 1.0}, {1.0, 0.0, 0.0, 1.0}}, eF[4][4] = {};
  const int row0 = w < kPair ? w : 0;  // first row of the wavefront's cells
  const bool gn_wave = kCh == 2 && w == 7;
  if (w < kPair || gn_wave) {
    const int ci = valid ? i : 0;
#pragma unroll
    for (int r = 0; r < (kCh == 2 ? kPair : 1); ++r) {
      if (r > 0 && !gn_wave) continue;
      const size_t cc = (size_t)clampi(jb + row0 + r, 0, P.ny - 1) * P.nx + ci;
      if (valid) {
#pragma unroll
        for (int k = 0; k < 4; ++k) eWn[r][k] = W[4 * cc + k];
      }
    }
    if (!kFill && w < kPair) {
      // the fluxes through the cell's left and right x faces and its lower and upper y faces
      const int jr = clampi(jb + w, 0, P.ny - 1);
      const UGKS_GLOBAL double* fl = recx + (size_t)R_FX * nfx + (size_t)jr * (P.nx + 1) + ci;
      const UGKS_GLOBAL double* fb = recy + (size_t)R_FX * nfy + (size_t)jr * P.nx + ci;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        eF[0][k] = fl[k * nfx];
        eF[1][k] = fl[k * nfx + 1];
        eF[2][k] = fb[k * nfy];
        eF[3][k] = fb[k * nfy + P.nx];
      }
    }
  }
  // face units of this wavefront: [fu0, fu1), all of both halves but the first half of the last
  // (wavefront 2 of four) or the second half of the first (wavefront 3 of four)
  constexpr int kUnits = kCh == 2 ? 1 : 3;
  const int fu0 = kCh == 2 ? w - kPair : (w == 2 ? 0 : 2);
  const bool face_wave = !kFill && w >= kPair && (kCh == 1 || w < 7);
  double flam[kUnits], fvel[kUnits];
  auto load_face_inputs = [&]() {
    if (!face_wave) return;
#pragma unroll
    for (int n = 0; n < kUnits; ++n) {
      const int u = fu0 + n;
      if (u < kPair) {
        const UGKS_GLOBAL double* rec = recx +
                                        (size_t)clampi(jb + u, 0, P.ny - 1) * (P.nx + 1) +
                                        clampi(i0 - kHalo + lane, 0, P.nx);
        flam[n] = rec[(size_t)R_LAM * nfx];
        fvel[n] = rec[(size_t)R_VY * nfx];
      } else {
        const UGKS_GLOBAL double* rec = recy + (size_t)clampi(jb + u - kPair, 0, P.ny) * P.nx +
                                        clampi(i0 - kHalo + lane, 0, P.nx - 1);
        flam[n] = rec[(size_t)R_LAM * nfy];
        fvel[n] = rec[(size_t)R_VY * nfy];
      }
    }
  };
  if constexpr (sizeof(T) == 8) load_face_inputs();
  // the records of the pair's faces: x faces i0-2 .. i0+62 of both rows, y face rows
  // jb .. jb+2 below / above lanes 0..63; indices clamped into the mesh for lanes and rows
  // outside it.  Every thread issues all its record loads before it uses any: one trip of a
  // load-then-store loop per value would wait out one memory latency per trip.
  constexpr int kThreads = kWave * kQuads * kCh;  // the launch's workgroup size
  constexpr int kNX = kPair * (kWave + 1) * kSF, kNY = (kPair + 1) * kWave * kSF;
  constexpr int kItX = kFill ? 1 : (kNX + kThreads - 1) / kThreads;
  constexpr int kItY = kFill ? 1 : (kNY + kThreads - 1) / kThreads;
  T vx[kItX], vy[kItY];
  if constexpr (!kFill) {
    auto fld_of = [](int s) { return s <= sf(R_UX) ? R_GC + s : R_GC + s + 1; };  // skip R_VY
#pragma unroll
    for (int it = 0; it < kItX; ++it) {
      const int e = threadIdx.x + it * kThreads;
      if (e < kNX) {
        const int r = e / ((kWave + 1) * kSF), rem = e - r * ((kWave + 1) * kSF);
        const int s = rem / (kWave + 1), fc = rem - s * (kWave + 1);  // faces fastest
        const int fi = clampi(i0 - kHalo + fc, 0, P.nx);
        const int row = clampi(jb + r, 0, P.ny - 1);
        vx[it] = T(recx[(size_t)fld_of(s) * nfx + (size_t)row * (P.nx + 1) + fi]);
      }
    }
#pragma unroll
    for (int it = 0; it < kItY; ++it) {
      const int e = threadIdx.x + it * kThreads;
      if (e < kNY) {
        const int r = e / (kWave * kSF), rem = e - r * (kWave * kSF);
        const int s = rem / kWave, fc = rem - s * kWave;  // faces fastest
        const int fi = clampi(i0 - kHalo + fc, 0, P.nx - 1);
        const int row = clampi(jb + r, 0, P.ny);
        vy[it] = T(recy[(size_t)fld_of(s) * nfy + (size_t)row * P.nx + fi]);
      }
    }
  }
  auto store_records = [&]() {
#pragma unroll
    for (int it = 0; it < kItX; ++it) {
      const int e = threadIdx.x + it * kThreads;
      if (e < kNX) {
        const int r = e / ((kWave + 1) * kSF), rem = e - r * ((kWave + 1) * kSF);
        const int s = rem / (kWave + 1), fc = rem - s * (kWave + 1);
        st.sx[r][s][fc] = vx[it];
      }
    }
#pragma unroll
    for (int it = 0; it < kItY; ++it) {
      const int e = threadIdx.x + it * kThreads;
      if (e < kNY) {
        const int r = e / (kWave * kSF), rem = e - r * (kWave * kSF);
        const int s = rem / kWave, fc = rem - s * kWave;
        st.sy[r][s][fc] = vy[it];
      }
    }
  };
  // FP32 storage has no registers to hold its share of the records through its part
  if constexpr (!kFill && sizeof(T) == 4) {
    store_records();
    load_face_inputs();
  }
  const double hstep = P.dv;
  // A start value below the normal range cannot be carried up to a peak that lies beyond the
  // chunk's first node: such a state (speed ratio |V| lambda^(1/2) above about 26 across v)
  // is flagged.
  bool lost = false;
  // the first v node of this workgroup's chunk in half h (h = 0: v >= 0, walked upwards)
  int vfirst[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const Half hv = axis_half(P.M, h == 0 ? 1 : -1, false);
    int c0, c1;
    chunk_range(hv.count, gv, Gv, c0, c1);
    vfirst[h] = hv.first + c0 * hv.step;
  }
  // Gauss start of exp(-lam (v - c)^2) at that node and its ratio to the next (FP64, stored
  // in the stage's type)
  auto start = [&](double lam, double c, int h, T* e, T* r, int col) {
    const double v0 = ((const UGKS_CONST double*)P.vm)[vfirst[h]];
    const double hs = h == 0 ? hstep : -hstep;
    const double d = v0 - c;
    const double x = lam * d * d;
    e[col] = T(exp(-x));
    r[col] = T(exp(-lam * hs * (2.0 * d + hs)));
    lost = lost || (x > 700.0 && (h == 0 ? c > v0 : c < v0));
  };
  // Gauss starts of g^n of the cells of row jb + r from their primitive state p
  auto start_gn = [&](const Prim& p, int r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) start(p.lam, p.V, h, st.gs[h][r][0][0], st.gs[h][r][0][1], lane);
  };
  if (w < kPair) {
    // Eq. (4) for row jb + w, and the cell's Maxwellians of W^n and W^{n+1} with the
    // weights of Eq. (3) solved for f^{n+1}: f1 = Af f + AdF dF + (A1 g^{n+1} + An g^n)
    const int r = w;
    const int jr = clampi(jb + r, 0, P.ny - 1);
    const bool mine = valid && (r == 0 ? store0 : true);
    const int ci = valid ? i : 0;
    const size_t cc = (size_t)jr * P.nx + ci;
    double Wn[4], W1[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) Wn[k] = eWn[0][k];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (kFill) {  // the ghost states of the current W
        W1[k] = Wn[k];
      } else {
        const double dW = (eF[0][k] - eF[1][k] + eF[2][k] - eF[3][k]) / P.area;
        W1[k] = valid ? Wn[k] + dW : Wn[k];
      }
    }
    // every velocity chunk of the segment forms the same W^{n+1}; chunk 0 stores it
    if (!kFill && mine && gg == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) Wout[4 * cc + k] = W1[k];
    }
    if (!kFill && P.adaptive && gg == 0) {
      // the adaptive step of the next step: the largest rate over the cells of W^{n+1}
      double rate = 0.0;
      if (mine)
        rate = (P.umax + fabs(W1[1] / W1[0])) / P.dx + (P.vmax + fabs(W1[2] / W1[0])) / P.dy;
      rate = wave_max(rate);
      if (lane == 0)
        atomicMax((unsigned long long*)(P.rmax + (parity ^ 1)),
                  (unsigned long long)__double_as_longlong(rate));
    }
    // the simulated time advances by this step's dt (one thread of the instance)
    if (!kFill && b == 0 && w == 0 && lane == 0)
      *P.tsum += step_dt(P, parity);
    Prim pn{}, p1{};
    double Af = 1.0, AdF = 1.0 / P.area, A1 = 0.0, An = 0.0;
    if (!P.collisionless) {
      const bool ok = prim_of(Wn, pn, P.lam_c) && prim_of(W1, p1, P.lam_c);
      if (!ok && mine) *P.flag = 1;
      const double tn = collision_time(pn, P.mu_ref), t1 = collision_time(p1, P.mu_ref);
      const double hdt = 0.5 * step_dt(P, parity);
      const double den = 1.0 / (1.0 + hdt / t1);
      Af = (1.0 - hdt / tn) * den;
      AdF = den / P.area;
      A1 = (p1.rho * p1.lam / kPi) * (hdt / t1) * den;
      An = (pn.rho * pn.lam / kPi) * (hdt / tn) * den;
      if (hpart) {  // the equilibrium of H: dof/(2 lambda) times that of G
        A1 *= (double)P.dof / (2.0 * p1.lam);
        An *= (double)P.dof / (2.0 * pn.lam);
      }
    }
    // A channel's ghost column (lane of cell -1 or nx) takes the ghost state of step n + 1,
    // formed from W^{n+1} of the cell next to it (Sec. 3.A), as its g^{n+1} with weight one
    // and every other Eq. (3) weight zero: the loop then writes the ghost Maxwellian of the
    // next step into the ghost column of f^{n+1}.  The first velocity chunk stores its W.
    // (both shifts run on every lane: a lane exchange inside a per-lane branch would read
    // the lanes the branch switched off)
    double Wc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double up = from_upper(W1[k]), dn = from_lower(W1[k]);
      Wc[k] = i < 0 ? up : dn;
    }
    if (ghost_w) {
      const int side = i < 0 ? 0 : 1;
      Prim pc;
      (void)prim_of(Wc, pc, P.lam_c);  // an invalid cell state is flagged by its own lane
      p1 = ghost_prim(P, side, jr, pc);
      pn = p1;
      if (gg == 0 && (r == 0 ? store0 : true))
        store_wg(I->Wg + 4 * ((size_t)side * P.ny + jr), p1, P.lam_c);
      Af = 0.0;
      AdF = 0.0;
      An = 0.0;
      A1 = p1.rho * p1.lam / kPi;
      if (hpart) A1 *= (double)P.dof / (2.0 * p1.lam);
    }
    if constexpr (kShak) {
      // heat flux of f^n about U^n from the cell's raw moments (moment kernel, chunk 0)
      const size_t nc = (size_t)P.nc;
      const UGKS_GLOBAL double* cm = I->hs + cell_sum_at(P, 0) + cc;
      double m[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) m[k] = valid ? cm[(size_t)k * nc] : 0.0;
      double qn[2];
      heat_flux(m[0], m[1], m[2], m[3], m[4], m[5], m[6], m[7], m[3] + m[5], pn.U, pn.V, qn);
      // no Shakhov factor on a ghost Maxwellian
      const double kn = P.collisionless || ghost_w ? 0.0 : P.pr_c * pn.lam * pn.lam / pn.rho;
      const double k1 = P.collisionless || ghost_w ? 0.0 : P.pr_c * p1.lam * p1.lam / p1.rho;
      sk[r][0][lane] = T(kn * qn[0]);
      sk[r][1][lane] = T(kn * qn[1]);
      sk[r][2][lane] = T(k1 * qn[0]);
      sk[r][3][lane] = T(k1 * qn[1]);
    }
    const double cell[C_COUNT] = {pn.lam, pn.U, pn.V, p1.lam, p1.U, p1.V, An, A1, Af, AdF};
#pragma unroll
    for (int n = 0; n < C_COUNT; ++n) st.cell[r][n][lane] = T(cell[n]);
    if constexpr (!kOwnQ) {
      qg[r][0][lane] = second_factor<T>(hstep, pn.lam);
      qg[r][1][lane] = second_factor<T>(hstep, p1.lam);
    }
    // Gauss starts of this cell in both halves of v
#pragma unroll
    for (int h = 0; h < 2; ++h)
      start(p1.lam, p1.V, h, st.gs[h][r][1][0], st.gs[h][r][1][1], lane);
    if constexpr (kCh == 1) start_gn(pn, r);
  } else if (gn_wave) {
    // g^n of both rows' cells; a ghost column's g^n has weight zero, so any finite state serves
#pragma unroll
    for (int r = 0; r < kPair; ++r) {
      Prim pn{};
      if (!P.collisionless) (void)prim_of(eWn[r], pn, P.lam_c);
      start_gn(pn, r);
    }
  } else if (face_wave) {
    // Gauss starts of the face units (FP64 records).  The last face of an x row (the right
    // face of lane 63) starts nothing: no written cell takes a flux from it.
#pragma unroll
    for (int n = 0; n < kUnits; ++n) {
      const int u = fu0 + n;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (kCh == 1 && ((w == 2 && n == 2 && h == 1) || (w == 3 && n == 0 && h == 0))) continue;
        T* e = u < kPair ? st.xs[h][u][0] : st.ys[h][u - kPair][0];
        T* r = u < kPair ? st.xs[h][u][1] : st.ys[h][u - kPair][1];
        start(flam[n], fvel[n], h, e, r, lane);
        if (h == 0)
          (u < kPair ? st.qx[u] : st.qy[u - kPair])[lane] = second_factor<T>(hstep, flam[n]);
      }
    }
  }
  if constexpr (!kFill && sizeof(T) == 8) store_records();
  if (lost && (valid || ghost_w)) *P.flag = 1;
  __syncthreads();
  // the workgroup's chunks kCh g .. kCh g + kCh - 1 of the quadrant's kCh G chunks
  const int sv = quad_sv(q);
  if constexpr (kFill) {
    if (quad_su(q) > 0)
      ghost_fill_quadrant<S, 1>(P, st, qg, lane, sv, jb, store0, kCh * g + c, kCh * G, gv, Gv,
                                ghost_w, fout, i);
    else
      ghost_fill_quadrant<S, -1>(P, st, qg, lane, sv, jb, store0, kCh * g + c, kCh * G, gv, Gv,
                                 ghost_w, fout, i);
    return;
  }
  if (quad_su(q) > 0)
    pair_quadrant<S, 1, kShak, kNode, kOwnQ>(P, st, qg, sk, lane, sv, jb, store0, kCh * g + c,
                                             kCh * G, gv, Gv, valid || ghost_w, ghost_lane,
                                             kCh == 2 && c == 1, fin, fout, i);
  else
    pair_quadrant<S, -1, kShak, kNode, kOwnQ>(P, st, qg, sk, lane, sv, jb, store0, kCh * g + c,
                                              kCh * G, gv, Gv, valid || ghost_w, ghost_lane,
                                              kCh == 2 && c == 1, fin, fout, i);
}

// Velocity chunks per update workgroup, kCh (its wavefronts: four quadrants times kCh), which
// share one stage, and the update waves per SIMD.  FP64: the registers of two rows allow two
// waves per SIMD; with two chunks, one workgroup of eight waves per CU, and sharing the stage
// halves its cost per velocity node; one chunk, two workgroups of four waves per CU (79.7 KB
// each, 81.8 Shakhov), serves meshes too small to give every CU a workgroup of two.  FP32 storage:
// four waves per SIMD, four workgroups of four waves per CU (39.9 KB each); the Shakhov form two
// waves per SIMD.
template <typename S, bool kShak>
constexpr int kUpdateWaves = sizeof(S) == 8 || kShak ? 2 : 4;

template <typename S, int kCh>
__global__ __launch_bounds__(kWave* kQuads* kCh)
__attribute__((amdgpu_waves_per_eu(kUpdateWaves<S, false>)))
void update_kernel(const Inst* inst, const int* off, int ninst, int step) {
  update_body<S, false, kCh>(inst, off, ninst, step);
}

// The chunks of this form split a quadrant's nodes instead of its u lines (update_by_node).  A
// kernel of its own: it takes a few registers more, and in FP32 storage spills two of them (12 bytes
// of scratch a lane), which would cost the solvers that take whole lines (400 x 100 x 40^2: 181 us
// without, 188 us with it).
template <typename S, int kCh>
__global__ __launch_bounds__(kWave* kQuads* kCh)
__attribute__((amdgpu_waves_per_eu(kUpdateWaves<S, false>)))
void update_kernel_nodes(const Inst* inst, const int* off, int ninst, int step) {
  update_body<S, false, kCh, false, true>(inst, off, ninst, step);
}

template <typename S, int kCh>
__global__ __launch_bounds__(kWave* kQuads* kCh)
__attribute__((amdgpu_waves_per_eu(kUpdateWaves<S, true>)))
void update_kernel_shakhov(const Inst* inst, const int* off, int ninst, int step) {
  update_body<S, true, kCh>(inst, off, ninst, step);
}

// The update kernel's fill mode (any collision model: a ghost Maxwellian carries no Shakhov
// factor), launched with the workgroups of the update kernel.
template <typename S, int kCh>
__global__ __launch_bounds__(kWave* kQuads* kCh)
__attribute__((amdgpu_waves_per_eu(kUpdateWaves<S, false>)))
void ghost_fill_kernel(const Inst* inst, const int* off, int ninst, int step) {
  update_body<S, false, kCh, true>(inst, off, ninst, step);
}

// ================================================================== host images
// The canonical host layout of f ([cell][velocity], doubles) and the velocity planes differ by a
// transpose, which runs here on 64 x 64 tiles in LDS: planes are read or written in 64 cells of
// a row, the host image (pinned memory, accessed over the host link) in 64 velocities of a
// cell, 512 contiguous bytes each way.  Bound by the host link and the host's copy to or from the
// caller's buffer: reading and setting the state of 80 x 40 cells at 29^2 (21.5 MB) takes 1.6 ms
// with a step on either side, 13.8 ms when the host did the transpose.  The piece: cells
// [c0, c0 + ncell) by velocities [v0, v0 + nvel) of the NC NV values of a cell, at
// img[(c - c0) nvel + v - v0].
constexpr int kTile = 64;
template <typename S, bool kOut>
__global__ __launch_bounds__(256) void state_kernel(UGKS_GLOBAL S* f, KParams P, long long c0,
                                                    int ncell, int v0, int nvel,
                                                    UGKS_GLOBAL double* img) {
  __shared__ double tile[kTile][kTile + 1];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  const int cb = blockIdx.x * kTile, vb = blockIdx.y * kTile;  // first cell and velocity
  const bool has_c = cb + lane < ncell, has_v = vb + lane < nvel;
  const long long c = c0 + cb + (has_c ? lane : 0);
  const int j = (int)(c / P.nx), i = (int)(c - (long long)j * P.nx);
  const int at = pidx(P, i, j);
  if constexpr (kOut) {
#pragma unroll 4
    for (int r = w; r < kTile; r += 4)
      if (has_c && vb + r < nvel) tile[r][lane] = ldv(plane_of(f, P, v0 + vb + r), at);
    __syncthreads();
#pragma unroll 4
    for (int r = w; r < kTile; r += 4)
      if (has_v && cb + r < ncell) img[(long long)(cb + r) * nvel + vb + lane] = tile[lane][r];
  } else {
#pragma unroll 4
    for (int r = w; r < kTile; r += 4)
      if (has_v && cb + r < ncell) tile[lane][r] = img[(long long)(cb + r) * nvel + vb + lane];
    __syncthreads();
#pragma unroll 4
    for (int r = w; r < kTile; r += 4)
      if (has_c && vb + r < nvel) stv(plane_of(f, P, v0 + vb + r), at, tile[r][lane]);
  }
}

// (rho, U, V, T) of n cells from their W into pinned host memory, two values a thread so that a
// wavefront's store is 1 KB of contiguous memory.  *bad becomes 1 if a cell's state is invalid
// or an invalid state was flagged.  One launch takes the place of two copies through the
// runtime's own staging and a host loop: one step and the moments of 40 x 10 cells (24^2) went
// from 63 to 44 us, ten steps and those of 400 x 100 (40^2) from 5.68 to 5.48 ms.
__global__ __launch_bounds__(256) void moments_kernel(const UGKS_GLOBAL double* W, int n,
                                                      double lam_c,
                                                      const UGKS_GLOBAL int* flag,
                                                      UGKS_GLOBAL double* out,
                                                      UGKS_GLOBAL int* bad) {
#pragma clang fp contract(off)
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int c = e >> 1;
  if (c >= n) return;
  const double rho = W[4 * (size_t)c], U = W[4 * (size_t)c + 1] / rho;
  const double V = W[4 * (size_t)c + 2] / rho;
  const double T = (W[4 * (size_t)c + 3] - 0.5 * rho * (U * U + V * V)) / (lam_c * rho);
  typedef double d2 __attribute__((ext_vector_type(2)));
  const d2 v = e & 1 ? d2{V, T} : d2{rho, U};
  *(UGKS_GLOBAL d2*)(out + 2 * (size_t)e) = v;
  if (!(rho > 0.0) || !(T > 0.0) || !isfinite(U) || !isfinite(V) || !isfinite(T) ||
      (e == 0 && *flag != 0))
    *bad = 1;
}

}  // namespace

// ================================================================== launchers
// Moment-kernel workgroups that a solver's velocity chunks aim for: 3 per CU.
constexpr long long kFillWorkgroups = 256 * 3;

int velocity_chunks(int nx, int ny, int K, int NC) {
  const long long base = (long long)((nx + kTileU - 1) / kTileU) * ny * NC;
  long long G = kFillWorkgroups / base;
  const int half = K / 2;  // nodes of the smaller half of the u axis
  if (G > half) G = half;
  if (G > 16) G = 16;
  return G < 1 ? 1 : (int)G;
}

// Velocity chunks per quadrant of the update kernel, U, for `base` workgroups per chunk and
// `slots` workgroups that run at once.  The update kernel adds nothing across chunks, so its
// chunks do not change any result.
//
// A batch of instances (update_chunks): the fewest chunks whose workgroups fill every round of
// the slots that they start to at least 85%, and at least one full round; at most 16.
int update_chunks(long long base, long long slots) {
  for (int U = 1; U <= 16; ++U) {
    const long long n = base * U;
    const long long rounds = (n + slots - 1) / slots;
    if (n >= slots && n * 100 >= 85 * rounds * slots) return U;
  }
  return 16;
}

// One instance (update_chunks_single): U, at most `cap` and 16, that minimises
// rounds x (2 + u nodes per chunk / vs), with `per_wg` chunks to a workgroup over the `half`
// u nodes of the smaller half and the v range in `vs` chunks: a workgroup's fixed cost (its
// stage and Gauss starts) counts as two u nodes of a whole v half; of equal costs the most
// workgroups.  On the paper's meshes and the 400x100 channel it picks the fastest U of a
// sweep or one within 1% of it.
int update_chunks_single(long long base, long long slots, int cap, int per_wg, int half,
                         int vs) {
  int best = 1;
  long long best_cost = -1;
  for (int U = 1; U <= cap && U <= 16; ++U) {
    const long long rounds = (base * U + slots - 1) / slots;
    const long long chunks = (long long)per_wg * U;
    const long long cost = rounds * (2LL * vs + (half + chunks - 1) / chunks);
    if (best_cost < 0 || cost <= best_cost) {
      best = U;
      best_cost = cost;
    }
  }
  return best;
}

// Whether the update kernel's G chunks of a quadrant split its nodes evenly (by node) rather than
// its u lines: K u nodes and vh v nodes of the longer halves, the latter one of Gv chunks, ch chunks
// to a workgroup.  The longest chunk sets the time, counted in nodes of the v loop, with four for
// every line it touches (its cubics and u Gaussians).  Of the two chunks of a workgroup, which share
// a SIMD, their mean counts, except where v is in chunks as well: these are short and wait for
// latency more than for one another, so a bound of the longest single one counts, a sixth of a node
// for each run past inside a line included.  On 129 solvers (20..400 x 10..100 cells, 8..101 nodes
// an axis, both storage types, H, periodic boxes) a step then takes 0.12% more than with the better
// of the two forms, at most 1.8%; always whole lines 1.1% and at most 17%, always by node 0.7% and
// 5%, with the bound of single chunks everywhere 0.33% and 4.8%.
// Steps by line and by node: 80 x 40 x 49^2, 25 lines over 12 chunks, 92.3 and 88.1 us; 200 x 50 x
// 101^2, 51 over 10, 938 and 911; 120 x 60 x 29^2 in FP32 storage, 15 over 14, 64.0 and 61.3.
bool update_by_node(int K, int vh, int Gv, int G, int ch) {
  constexpr int NB = 3, kLine = 4;  // nodes of a group, of a line's setup
  const int lines = K - K / 2, vg = (vh + NB - 1) / NB;
  if (Gv > 1) {
    const int len = (lines * vg + G - 1) / G;  // groups
    const int touched = len > 1 ? (len - 2) / vg + 2 : 1;
    return 6 * (NB * len + kLine * touched) + vh < 6 * ((lines + G - 1) / G) * (vh + kLine);
  }
  auto nodes = [&](int group) { return group / vg * vh + std::min(group % vg * NB, vh); };
  int whole = 0, split = 0;  // of the longest workgroup
  for (int g = 0; g < G; g += ch) {
    int w = 0, s = 0;
    for (int c = g; c < g + ch; ++c) {
      int a0, a1;
      chunk_range(lines, c, G, a0, a1);
      w += (a1 - a0) * (vh + kLine);
      chunk_range(lines * vg, c, G, a0, a1);
      if (a1 > a0) s += nodes(a1) - nodes(a0) + ((a1 - 1) / vg - a0 / vg + 1) * kLine;
    }
    whole = std::max(whole, w);
    split = std::max(split, s);
  }
  return split < whole;
}

int update_vsplit(int nx, int ny, int K, int M, int NC, int fp32, int shak, int cap) {
  const long long base = (long long)((nx + kTileU - 1) / kTileU) * ((ny + 1) / 2) * NC;
  const int umax = std::max(1, std::min(K / 2, 16));
  // four-wavefront workgroups that run at once: 256 CUs x update waves per SIMD
  const long long slots = 256LL * (fp32 ? (shak ? kUpdateWaves<float, true>
                                                 : kUpdateWaves<float, false>)
                                         : kUpdateWaves<double, false>);
  if (2 * base * umax >= slots) return 1;
  int vs = (int)(slots / (base * umax));
  vs = std::min(vs, (M / 2) / 4);
  if (cap > 0) vs = std::min(vs, cap);
  return std::max(vs, 1);
}

size_t plan_bytes(int n) {
  const size_t inst = ((sizeof(Inst) * (size_t)n + 255) / 256) * 256;
  return inst + 6 * (((size_t)(n + 1) * sizeof(int) + 255) / 256) * 256;
}

PlanTotals build_plan(const Inst* insts, int n, void* buf, const void* dev, PlanView* view) {
  char* h = static_cast<char*>(buf);
  const char* d = static_cast<const char*>(dev);
  const size_t inst_bytes = ((sizeof(Inst) * (size_t)n + 255) / 256) * 256;
  const size_t off_bytes = (((size_t)(n + 1) * sizeof(int) + 255) / 256) * 256;
  // The instances with the longest workgroups first (their nodes per quadrant), so that a launch
  // ends on short ones.  Twelve FP32-storage solves of the serving shapes (190M updates a step):
  // 1174 us in the callers' order with one XCD range over all instances, 1022 with the range per
  // instance (some XCDs had only long workgroups), 949 with this order as well.  More and smaller
  // chunks for the longer instances gained nothing further.
  Inst* img = reinterpret_cast<Inst*>(h);
  {
    std::unique_ptr<int[]> order(n > 1 ? new (std::nothrow) int[n] : nullptr);
    if (order) {
      for (int q = 0; q < n; ++q) order[q] = q;
      auto nodes = [&](int q) { return (long long)insts[q].P.K * insts[q].P.M; };
      std::sort(order.get(), order.get() + n, [&](int a, int b) {
        return nodes(a) != nodes(b) ? nodes(a) > nodes(b) : a < b;
      });
    }
    for (int q = 0; q < n; ++q) std::memcpy(img + q, insts + (order ? order[q] : q), sizeof(Inst));
    insts = img;
  }
  int* off[6];
  for (int a = 0; a < 6; ++a) off[a] = reinterpret_cast<int*>(h + inst_bytes + a * off_bytes);
  PlanTotals t{};
  // each instance keeps the velocity chunks it was created with, in any plan, so that its
  // sums are added in the same order whether it is stepped alone or in a batch
  long long upd_base = 0;  // update workgroups of all instances with one chunk
  for (int q = 0; q < n; ++q) {
    const KParams& P = insts[q].P;
    upd_base += (long long)((P.nx + kTileU - 1) / kTileU) * ((P.ny + 1) / 2) * P.NC * P.vsplit;
  }
  // velocity chunks per update workgroup (FP64 two, FP32 storage one) and the workgroups
  // that run at once: 256 CUs x waves per CU / waves per workgroup
  const bool shak = n > 0 && insts[0].P.shak;
  const bool f32 = n > 0 && insts[0].fp32;
  const int waves = f32 ? (shak ? kUpdateWaves<float, true> : kUpdateWaves<float, false>)
                        : kUpdateWaves<double, false>;
  int per_wg = f32 ? 1 : 2;
  // each workgroup's chunks take at least one u node each of the smaller half
  auto cap_of = [&](const KParams& P, int ch) {
    const int c = P.K / 2 / ch;
    return c < 1 ? 1 : c;
  };
  auto choose = [&](int ch) {
    const long long slots = 256LL * waves / ch;
    if (n == 1)
      return update_chunks_single(upd_base, slots, cap_of(insts[0].P, ch), ch, insts[0].P.K / 2,
                                  insts[0].P.vsplit);
    return update_chunks(upd_base, slots);
  };
  int U = choose(per_wg);
  // a mesh that leaves more than half the CUs without a workgroup of two chunks takes one
  // chunk per workgroup: twice the workgroups, on twice the CUs
  if (per_wg == 2 && n == 1 && upd_base * U < 128) {
    per_wg = 1;
    U = choose(1);
  }
  t.upd_ch = per_wg;
  for (int q = 0; q < n; ++q) {
    img[q].gsplit = insts[q].P.gmax;
    const int cap = cap_of(insts[q].P, per_wg);
    img[q].usplit = U < cap ? U : cap;
  }
  // a batch's chunks are few and long: whole lines
  if (n == 1 && !shak) {
    const KParams& P = insts[0].P;
    const int vh = ((P.M - P.M / 2) + P.vsplit - 1) / P.vsplit;
    t.upd_nodes = update_by_node(P.K, vh, P.vsplit, per_wg * img[0].usplit, per_wg) ? 1 : 0;
  }
  // Faces and wavefronts per workgroup of the chunked interface kernel: 16 or 32 faces while each
  // workgroup (eight wavefronts, whose registers fill a CU) still has a CU of its own, then 64,
  // with four wavefronts where even those would be more than one to a CU.
  long long wide = 0;
  for (int q = 0; q < n; ++q) {
    const KParams& P = insts[q].P;
    if (img[q].gsplit * P.NC > 1) wide += P.ny * (P.nx + 1LL) + (P.ny + 1LL) * P.nx;
  }
  t.red_faces = wide <= 250 * 16 ? 16 : (wide <= 250 * 32 ? 32 : 64);
  t.red_waves = wide <= 250 * 64 ? 8 : 4;
  for (int q = 0; q < n; ++q) {
    const KParams& P = insts[q].P;
    const int G = img[q].gsplit * P.NC;  // chunks of G, then those of H
    const int nfx = P.ny * (P.nx + 1), nfy = (P.ny + 1) * P.nx;
    off[0][q] = t.sums;
    off[1][q] = t.upd;
    off[2][q] = t.face;
    off[3][q] = t.ghost;
    off[4][q] = t.red;
    off[5][q] = 0;
    t.shak = t.shak || P.shak;
    t.sums += ((P.nx + kTileS - 1) / kTileS) * P.ny * G;
    t.upd += ((P.nx + kTileU - 1) / kTileU) * ((P.ny + 1) / 2) * img[q].usplit * P.vsplit * P.NC;
    if (G > 1)
      t.red += (nfx + t.red_faces - 1) / t.red_faces + (nfy + t.red_faces - 1) / t.red_faces +
               (P.shak ? ((kSlotsShakhov - kSlotCell) * P.nc + kWave * t.red_waves - 1) /
                             (kWave * t.red_waves)
                       : 0);
    else
      t.face += (nfx + 255) / 256 + (nfy + 255) / 256;
    if (P.bc == UGKS_BC_CHANNEL) {
      t.channel = 1;
    } else {
      t.periodic = 1;
      t.ghost += ghost_blocks(P.nx) * P.NV * P.NC;
    }
  }
  off[0][n] = t.sums;
  off[1][n] = t.upd;
  off[2][n] = t.face;
  off[3][n] = t.ghost;
  off[4][n] = t.red;
  off[5][n] = 0;
  view->inst = reinterpret_cast<const Inst*>(d);
  view->off_sums = reinterpret_cast<const int*>(d + inst_bytes + 0 * off_bytes);
  view->off_upd = reinterpret_cast<const int*>(d + inst_bytes + 1 * off_bytes);
  view->off_face = reinterpret_cast<const int*>(d + inst_bytes + 2 * off_bytes);
  view->off_ghost = reinterpret_cast<const int*>(d + inst_bytes + 3 * off_bytes);
  view->off_red = reinterpret_cast<const int*>(d + inst_bytes + 4 * off_bytes);
  view->ninst = n;
  view->step = 0;
  return t;
}

hipError_t launch_poison(const PlanView& pv, int fp32, long long nvalues, hipStream_t s) {
  const unsigned blocks = (unsigned)((nvalues + 255) / 256);
  if (fp32)
    poison_kernel<float><<<blocks, 256, 0, s>>>(pv);
  else
    poison_kernel<double><<<blocks, 256, 0, s>>>(pv);
  return hipGetLastError();
}

hipError_t launch_init(const PlanView& pv, int fp32, long long nvalues, hipStream_t s) {
  const unsigned blocks = (unsigned)((nvalues + 255) / 256);
  if (fp32)
    init_kernel<float><<<blocks, 256, 0, s>>>(pv);
  else
    init_kernel<double><<<blocks, 256, 0, s>>>(pv);
  return hipGetLastError();
}

hipError_t launch_state(const KParams& P, void* f, int fp32, bool out, long long c0, int ncell,
                        int v0, int nvel, double* img, hipStream_t s) {
  const dim3 g((unsigned)((ncell + kTile - 1) / kTile), (unsigned)((nvel + kTile - 1) / kTile));
  float* f32 = static_cast<float*>(f);
  double* f64 = static_cast<double*>(f);
  if (fp32 && out)
    state_kernel<float, true><<<g, 256, 0, s>>>(gp(f32), P, c0, ncell, v0, nvel, gp(img));
  else if (fp32)
    state_kernel<float, false><<<g, 256, 0, s>>>(gp(f32), P, c0, ncell, v0, nvel, gp(img));
  else if (out)
    state_kernel<double, true><<<g, 256, 0, s>>>(gp(f64), P, c0, ncell, v0, nvel, gp(img));
  else
    state_kernel<double, false><<<g, 256, 0, s>>>(gp(f64), P, c0, ncell, v0, nvel, gp(img));
  return hipGetLastError();
}

hipError_t launch_moments(const double* W, int n, double lam_c, const int* flag, double* out,
                          int* bad, hipStream_t s) {
  moments_kernel<<<(unsigned)((2LL * n + 255) / 256), 256, 0, s>>>(
      gp(W), n, lam_c, gp(flag), gp(out), gp(bad));
  return hipGetLastError();
}

hipError_t launch_ghost_fill(const PlanView& pv, const PlanTotals& t, int fp32, hipStream_t s) {
  if (!t.channel) return hipSuccess;
  const unsigned nt = (unsigned)(kWave * kQuads * t.upd_ch);
  const Inst* in = pv.inst;
  const int ni = pv.ninst, st = pv.step;
  if (fp32)
    ghost_fill_kernel<float, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
  else if (t.upd_ch == 2)
    ghost_fill_kernel<double, 2><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
  else
    ghost_fill_kernel<double, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
  return hipGetLastError();
}

// phase 0 ghosts, 1 moment sums, 2 interface scalars, 3 cell update
hipError_t launch_phase(const PlanView& pv, const PlanTotals& t, int fp32, int phase,
                        hipStream_t s) {
  const Inst* in = pv.inst;
  const int ni = pv.ninst, st = pv.step;
  constexpr unsigned kSumWg = kWave * kQuads;
  switch (phase) {
    case 0:
      if (t.ghost == 0) return hipSuccess;  // no periodic instance
      if (fp32)
        ghost_kernel<float><<<(unsigned)t.ghost, kGhostThreads, 0, s>>>(in, pv.off_ghost, ni, st);
      else
        ghost_kernel<double><<<(unsigned)t.ghost, kGhostThreads, 0, s>>>(in, pv.off_ghost, ni, st);
      break;
    case 1:
      if (t.shak) {
        if (fp32)
          sums_kernel<float, true><<<(unsigned)t.sums, kSumWg, 0, s>>>(in, pv.off_sums, ni, st);
        else
          sums_kernel<double, true><<<(unsigned)t.sums, kSumWg, 0, s>>>(in, pv.off_sums, ni, st);
      } else {
        if (fp32)
          sums_kernel<float, false><<<(unsigned)t.sums, kSumWg, 0, s>>>(in, pv.off_sums, ni, st);
        else
          sums_kernel<double, false><<<(unsigned)t.sums, kSumWg, 0, s>>>(in, pv.off_sums, ni, st);
      }
      break;
    case 2:
      if (t.red > 0) {
        if (t.red_faces == 16)
          faces_kernel_chunks<16, 8><<<(unsigned)t.red, kWave * 8, 0, s>>>(in, pv.off_red, ni, st);
        else if (t.red_faces == 32)
          faces_kernel_chunks<32, 8><<<(unsigned)t.red, kWave * 8, 0, s>>>(in, pv.off_red, ni, st);
        else if (t.red_waves == 8)
          faces_kernel_chunks<64, 8><<<(unsigned)t.red, kWave * 8, 0, s>>>(in, pv.off_red, ni, st);
        else
          faces_kernel_chunks<64, 4><<<(unsigned)t.red, kWave * 4, 0, s>>>(in, pv.off_red, ni, st);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      if (t.face > 0) faces_kernel<<<(unsigned)t.face, 256, 0, s>>>(in, pv.off_face, ni, st);
      break;
    default: {
      // FP32 storage runs one chunk per workgroup (build_plan never asks for two)
      const unsigned nt = (unsigned)(kWave * kQuads * t.upd_ch);
      if (t.shak) {
        if (fp32)
          update_kernel_shakhov<float, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else if (t.upd_ch == 2)
          update_kernel_shakhov<double, 2><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else
          update_kernel_shakhov<double, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
      } else if (t.upd_nodes) {
        if (fp32)
          update_kernel_nodes<float, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else if (t.upd_ch == 2)
          update_kernel_nodes<double, 2><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else
          update_kernel_nodes<double, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
      } else {
        if (fp32)
          update_kernel<float, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else if (t.upd_ch == 2)
          update_kernel<double, 2><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
        else
          update_kernel<double, 1><<<(unsigned)t.upd, nt, 0, s>>>(in, pv.off_upd, ni, st);
      }
    }
  }
  return hipGetLastError();
}

hipError_t launch_step(const PlanView& pv, const PlanTotals& t, int fp32, hipStream_t s,
                       hipEvent_t* ev) {
  for (int phase = 0; phase < 4; ++phase) {
    if (ev) (void)hipEventRecord(ev[2 * phase], s);
    const hipError_t e = launch_phase(pv, t, fp32, phase, s);
    if (ev) (void)hipEventRecord(ev[2 * phase + 1], s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ugks
