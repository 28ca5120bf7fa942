// etics_jerk.hip -- the SCF jerk and the batched fourth-order Hermite integrator.
//
// The paper notes that Hernquist's SCF code computes the jerk, the time derivative of
// the force (Section 3.4), for its fourth-order Hermite scheme, and names that scheme
// as the next integrator for SCF (Section 5.4; not for MEX, whose force derivative is
// discontinuous at shell crossings).  Here the jerk of particle i is the total time
// derivative of its acceleration when every particle moves with its velocity:
//   j_i = d/dt a(x_i + v_i t; A(t), B(t)) at t = 0,
// with dA/dt, dB/dt from etics_coeff_dot.hip.  The synthesis of etics_force_synth.hpp
// runs on Dual numbers (value, time derivative): the field point carries its velocity
// and each prepared coefficient its time derivative, so the one pass returns a and j.
//
// Hermite predictor-corrector (Makino & Aarseth 1992), one shared step dt per call:
//   predict  x_p = x + v dt + a dt^2/2 + j dt^3/6,   v_p = v + a dt + j dt^2/2,
//   evaluate a_1, j_1 at (x_p, v_p)  (coefficients and their derivatives there),
//   correct  v_1 = v + (a + a_1) dt/2 + (j - j_1) dt^2/12,
//            x_1 = x + (v + v_1) dt/2 + (a - a_1) dt^2/12.
// The jerk kernel applies the corrector to its particle as soon as a_1, j_1 are known,
// and (except in the last step) the next step's predictor, so a step is: coefficients
// and their derivatives at the predicted state, two reductions, the coefficient
// rescale and the jerk pass.  Steps 1 .. nsteps-1 are captured once into a hipGraph
// and replayed, the last step runs directly (as the leapfrog in etics_batched.hip).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>

#include "etics_device.hpp"
#include "etics_force_synth.hpp"
#include "etics_internal.hpp"

namespace etics {

// ---------------------------------------------------------------- coefficient prep
// FP64: prepared coefficients with their time derivatives, Dual [4K] per system, the
// same scaling as the force pass (Hernquist-Ostriker basis); FP32: the force pass's own
// preparation (etics_force.hip), for the matrix cores.
//   [0,K)   (su A, su dA/dt)   [K,2K)  (su B, su dB/dt)
//   [2K,3K) (sw A, sw dA/dt)   [3K,4K) (sw B, sw dB/dt)
__global__ __launch_bounds__(256) void scf_jerk_prep_kernel(const double* __restrict__ A,
                                                           const double* __restrict__ B,
                                                           const double* __restrict__ Ad,
                                                           const double* __restrict__ Bd, int nmax,
                                                           int lmax, int nsys, Dual<double>* __restrict__ cf) {
  const int K = (nmax + 1) * (lmax + 1) * (lmax + 2) / 2;
  const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (g >= int64_t(nsys) * K) return;
  const int sys = int(g / K);
  const int k = int(g - int64_t(sys) * K);
  const int L2 = (lmax + 1) * (lmax + 2) / 2;
  const int n = k / L2;
  const int lm = k - n * L2;
  int l = 0;
  while ((l + 1) * (l + 2) / 2 <= lm) ++l;
  const double al = basis_alpha(kBasisHO, l);
  const double s4 = -2.0 * sqrt(kPi);
  const double su = s4 * gegen_k(n, al);
  const double sw = n >= 1 ? s4 * 2.0 * al * 2.0 * gegen_k(n - 1, al + 1.0) : 0.0;
  Dual<double>* c = cf + size_t(sys) * 4 * K;
  c[k] = Dual<double>(su * A[g], su * Ad[g]);
  c[K + k] = Dual<double>(su * B[g], su * Bd[g]);
  c[2 * K + k] = Dual<double>(sw * A[g], sw * Ad[g]);
  c[3 * K + k] = Dual<double>(sw * B[g], sw * Bd[g]);
}

size_t jerk_prep_bytes(int nmax, int lmax, int prec) {
  return prec == ETICS_FP64 ? size_t(8) * coeff_count(nmax, lmax) * 8 : size_t(2) * mm_offset(lmax + 1, nmax) * 4;
}

// ---------------------------------------------------------------- jerk pass
// What the jerk pass of a Hermite step does with a particle's a and j:
//   kStart:   store them as the state's a, j and predict the first step;
//   kStep:    correct the state with them, store them, predict the next step;
//   kLast:    correct the state with them and store them.
enum HermiteMode { kStart = 1, kStep = 2, kLast = 3 };

struct JerkArgs {
  const double *x, *y, *z, *vx, *vy, *vz;  // field points and their velocities
  int64_t n;
  const void* cf;                          // prepared Dual coefficients
  double *ax, *ay, *az, *jx, *jy, *jz;     // single system: outputs; Hermite: the state's a and j
  // Hermite state: positions and velocities corrected in place, and the predicted ones (the
  // field points of the next pass)
  double *sx, *sy, *sz, *svx, *svy, *svz;
  double *px, *py, *pz, *pvx, *pvy, *pvz;
  int K, nmax, lmax, mode;
  double dt;
};

// point i's acceleration and jerk o: to the outputs, or (HERMITE) where the mode says
template <typename S, bool HERMITE>
__device__ __forceinline__ void jerk_store(const JerkArgs& a, int64_t i, const ForceOut<Dual<S>>& o) {
  const double g[3] = {double(o.gx.v), double(o.gy.v), double(o.gz.v)};
  const double jk[3] = {double(o.gx.d), double(o.gy.d), double(o.gz.d)};
  double* A[3] = {a.ax, a.ay, a.az};
  double* J[3] = {a.jx, a.jy, a.jz};
  if constexpr (!HERMITE) {
    for (int c = 0; c < 3; ++c) {
      A[c][i] = g[c];
      J[c][i] = jk[c];
    }
    return;
  }
  double* X[3] = {a.sx, a.sy, a.sz};
  double* V[3] = {a.svx, a.svy, a.svz};
  double* P[3] = {a.px, a.py, a.pz};
  double* PV[3] = {a.pvx, a.pvy, a.pvz};
  const double dt = a.dt, h = 0.5 * dt, q = dt * dt / 12.0;
  // all reads before the first write: one wait for them instead of one per component
  double x[3], v[3], a0[3], j0[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    x[c] = X[c][i];
    v[c] = V[c][i];
    a0[c] = a.mode != kStart ? A[c][i] : 0.0;
    j0[c] = a.mode != kStart ? J[c][i] : 0.0;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (a.mode != kStart) {  // corrector with the step's starting a, j
      const double v1 = __builtin_fma(q, j0[c] - jk[c], __builtin_fma(h, a0[c] + g[c], v[c]));
      x[c] = __builtin_fma(q, a0[c] - g[c], __builtin_fma(h, v[c] + v1, x[c]));
      v[c] = v1;
      X[c][i] = x[c];
      V[c][i] = v[c];
    }
    A[c][i] = g[c];
    J[c][i] = jk[c];
    if (a.mode != kLast) {  // predictor of the next step
      P[c][i] = __builtin_fma(dt * dt * dt / 6.0, jk[c],
                              __builtin_fma(0.5 * dt * dt, g[c], __builtin_fma(dt, v[c], x[c])));
      PV[c][i] = __builtin_fma(0.5 * dt * dt, jk[c], __builtin_fma(dt, g[c], v[c]));
    }
  }
}

// FP64: point i, FMAs on coefficients read through the constant address space ([4][K]) or
// from LDS (QUAD: [K][4]).  No kernel loops over points here: the compiler moves the FP64
// constants out of such a loop, and the registers for them are not there (290 of them went to
// vector lanes at (8, 6)).  A single system, N = 10^6, with a loop / here, us a call: (8, 6) 413 /
// 395, (12, 12) 3670 / 2450, (20, 14) 8380 / 5570.
template <int LB, bool HERMITE, bool QUAD, typename CP>
__device__ __forceinline__ void jerk_point_f64(const JerkArgs& a, CP cf, int64_t i) {
  const auto s = sph_dual<double, kBasisHO, true>(a.x[i], a.y[i], a.z[i], a.vx[i], a.vy[i], a.vz[i]);
  RadialDual<CP, QUAD> rad{cf, a.K, a.nmax, a.lmax};
  jerk_store<double, HERMITE>(a, i, synth_point<Dual<double>, LB, true, kBasisHO>(s, rad, a.lmax));
}
// one system's prepared coefficients, [4][K], to the workgroup's LDS as [K][4]
__device__ __forceinline__ void jerk_coeffs_to_lds(const Dual<double>* cf, int K, Dual<double>* lds) {
  for (int i = threadIdx.x; i < 4 * K; i += blockDim.x) {
    const int which = i / K, idx = i - which * K;
    lds[4 * idx + which] = cf[i];
  }
  __syncthreads();
}
// Where a single system's FP64 coefficients are read from: LDS from lmax bucket 12 on, where
// the scalar loads' latency bounds the one wavefront a SIMD holds ((20, 14): 501 / 344 us a call
// at N = 10^4, 8.40 / 5.57 ms at 10^6); below, the LDS reads do at large N ((10, 10): 1.27 / 1.49
// ms at 10^6).
template <typename S, int LB>
constexpr bool kJerkLds = sizeof(S) == 8 && LB > 10;

// FP32: the radial sums on the matrix cores, which need every lane: the loop is uniform over
// the workgroup and a lane past the end computes a point at rest at the origin.  At (8, 6)
// a wavefront issues 3050 VALU and matrix instructions a point instead of 4600, which shows
// only once the memory traffic of the Hermite step (290 bytes a particle) is asked for in
// time: a lane's next point and the state to correct are read together, before any write.
// 256 systems, (8, 6), 4 steps: 8.96 -> 8.45 ms.
template <int LB>
__device__ __forceinline__ void jerk_points_mm(const JerkArgs& a, const float* cf, int64_t i0, int64_t i1,
                                               int64_t stride) {
  RadialMM<Dual<float>, true, kBasisHO> rad(cf, a.nmax, a.lmax);
  rad.template start<0>();
  double x, y, z, vx, vy, vz;
  auto load = [&](int64_t i) {
    const bool valid = i < i1;
    x = valid ? a.x[i] : 0.0;
    y = valid ? a.y[i] : 0.0;
    z = valid ? a.z[i] : 0.0;
    vx = valid ? a.vx[i] : 0.0;
    vy = valid ? a.vy[i] : 0.0;
    vz = valid ? a.vz[i] : 0.0;
  };
  load(i0 + threadIdx.x);
  for (; i0 < i1; i0 += stride) {
    const int64_t i = i0 + threadIdx.x;
    const auto s = sph_dual<float, kBasisHO, true>(x, y, z, vx, vy, vz);
    const auto o = synth_point<Dual<float>, LB, true, kBasisHO>(s, rad, a.lmax);
    // before the stores: loads and stores are waited for in order
    load(i + stride);
    rad.template start<0>();
    if (i < i1) jerk_store<float, true>(a, i, o);
  }
}

// A single system's points, one per lane and no loop over them: in a loop every array's address
// stayed in registers over the synthesis (48 of them, most of them in scratch).  N = 10^6, vector
// FMAs / matrix cores in a loop / here, us a call: (4, 4) 59 / 64 / 54, (8, 6) 142 / 165 / 116,
// (10, 10) 425 / 372 / 276, (20, 14) 2440 / 2470 / 936.
template <int LB>
__device__ __forceinline__ void jerk_point_mm(const JerkArgs& a, int64_t i) {
  RadialMM<Dual<float>, true, kBasisHO> rad(reinterpret_cast<const float*>(a.cf), a.nmax, a.lmax);
  rad.template start<0>();
  const bool valid = i < a.n;
  const auto s = sph_dual<float, kBasisHO, true>(valid ? a.x[i] : 0.0, valid ? a.y[i] : 0.0, valid ? a.z[i] : 0.0,
                                           valid ? a.vx[i] : 0.0, valid ? a.vy[i] : 0.0, valid ? a.vz[i] : 0.0);
  const auto o = synth_point<Dual<float>, LB, true, kBasisHO>(s, rad, a.lmax);
  if (valid) jerk_store<float, false>(a, i, o);
}

// Wavefronts a SIMD (the second launch bound), FP32: as many as the registers allow without
// scratch, or with little of it where that measured faster.  Single system, N = 10^6, us a
// call: (8, 6) 3 (52 bytes of scratch a lane) / 2 (none) 119 / 124; (10, 10) 2 / 1 276 / 376;
// (12, 12) 2 (128 bytes) / 1 (none) 414 / 548; (20, 14) 2 (460 bytes) / 1 (none) 870 / 939, but
// 78 / 65 at 10^4.  Batched, Hermite steps, ms: (8, 6) 3 (120 bytes) / 2 (none) 8.52 / 8.43;
// (12, 12) 2 (416 bytes) / 1 (none) 16.3 / 16.7; (20, 14) 2 (604 bytes) / 1 (none) 22.3 / 20.4.
template <typename S, int LB>
__global__ __launch_bounds__(256, sizeof(S) == 8 ? 1 : LB <= 6 ? 3 : LB <= 12 ? 2 : 1) void scf_jerk_kernel(const JerkArgs a) {
  extern __shared__ __align__(16) unsigned char jerk_lds[];
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if constexpr (sizeof(S) == 4) {
    jerk_point_mm<LB>(a, i);
  } else if constexpr (kJerkLds<S, LB>) {
    Dual<S>* lds_cf = reinterpret_cast<Dual<S>*>(jerk_lds);
    jerk_coeffs_to_lds(reinterpret_cast<const Dual<S>*>(a.cf), a.K, lds_cf);
    if (i < a.n) jerk_point_f64<LB, false, true>(a, (LdsPtr<Dual<S>>)(lds_cf), i);
  } else {
    if (i < a.n)
      jerk_point_f64<LB, false, false>(a, ConstPtr<Dual<S>>(reinterpret_cast<const Dual<S>*>(a.cf)), i);
  }
}

// batched systems: `split` (times gridDim.y) workgroups per unit of `unit` particles of one
// system, as the batched force kernel; FP64: the workgroup first copies its system's prepared
// coefficients to LDS as [K][4] and reads them as broadcast VGPR operands, and its part has at
// most one particle for each lane, so that there is no loop out of which the constants are moved
// (to vector lanes).  With a loop / here, 4 Hermite steps, ms: 128 systems (8, 6) 9.13 / 8.49,
// (20, 14) 78.6 / 73.4; 16 systems of 1000 (8, 6) 1.44 / 0.97.
template <typename S, int LB>
__global__ __launch_bounds__(256, sizeof(S) == 8 ? 1 : LB <= 4 ? 3 : LB <= 12 ? 2 : 1) void scf_jerk_batched_kernel(const JerkArgs a,
                                                               const int64_t* __restrict__ offsets,
                                                               const int* __restrict__ ustart,
                                                               const int* __restrict__ usys, int nsys,
                                                               int unit, int split) {
  extern __shared__ __align__(16) unsigned char jerk_lds[];
  const int u = blockIdx.x / split;
  const int part = blockIdx.x % split + split * blockIdx.y;
  if (u >= ustart[nsys]) return;
  const int sys = usys[u];
  int64_t b = offsets[sys], e = offsets[sys + 1];
  b = b < 0 ? 0 : (b > a.n ? a.n : b);
  e = e < b ? b : (e > a.n ? a.n : e);
  const int parts = split * gridDim.y;
  const int64_t kPart = (unit + parts - 1) / parts;
  const int64_t u0 = b + int64_t(u - ustart[sys]) * unit;
  const int64_t ue0 = u0 + unit < e ? u0 + unit : e;
  const int64_t ub = u0 + part * kPart < ue0 ? u0 + part * kPart : ue0;
  const int64_t ue = ub + kPart < ue0 ? ub + kPart : ue0;
  if constexpr (sizeof(S) == 4) {
    jerk_points_mm<LB>(a,
                       reinterpret_cast<const float*>(a.cf) +
                           size_t(__builtin_amdgcn_readfirstlane(sys)) * 2 * mm_offset(a.lmax + 1, a.nmax),
                       ub, ue, blockDim.x);
  } else {
    if (ub >= ue) return;
    Dual<S>* lds_cf = reinterpret_cast<Dual<S>*>(jerk_lds);
    jerk_coeffs_to_lds(reinterpret_cast<const Dual<S>*>(a.cf) + size_t(sys) * 4 * a.K, a.K, lds_cf);
    const int64_t i = ub + threadIdx.x;
    if (i < ue) jerk_point_f64<LB, true, true>(a, (LdsPtr<Dual<S>>)(lds_cf), i);
  }
}

namespace {

struct JerkBatch {
  const int64_t* offsets;
  const int* ustart;
  const int* usys;
  int nsys, unit, split;
};

template <typename S, int LBV>
void launch_jerk_kernel(const JerkArgs& a, int grid, const JerkBatch* bi, hipStream_t st) {
  // FP64 from LDS: 4 K Dual values, at the largest cutoffs 158 KiB; more than 64 KiB has to be
  // allowed first (failures surface at the launch)
  const size_t lds = sizeof(S) == 8 && (bi || kJerkLds<S, LBV>) ? size_t(4) * a.K * sizeof(Dual<S>) : 0;
  auto allow = [&](const void* kfn) {
    if (lds > 64 * 1024) (void)hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  };
  if (bi) {
    allow(reinterpret_cast<const void*>(scf_jerk_batched_kernel<S, LBV>));
    const int rows = sizeof(S) == 8 ? (bi->unit + 256 * bi->split - 1) / (256 * bi->split) : 1;
    hipLaunchKernelGGL((scf_jerk_batched_kernel<S, LBV>), dim3(grid, rows), dim3(256), lds, st, a, bi->offsets,
                       bi->ustart, bi->usys, bi->nsys, bi->unit, bi->split);
    return;
  }
  allow(reinterpret_cast<const void*>(scf_jerk_kernel<S, LBV>));
  // a grid holds less than 2^32 threads
  constexpr int64_t kMost = int64_t(1) << 30;
  for (int64_t at = 0; at < a.n; at += kMost) {
    JerkArgs b = a;
    b.n = a.n - at < kMost ? a.n - at : kMost;
    for (const double** p : {&b.x, &b.y, &b.z, &b.vx, &b.vy, &b.vz}) *p += at;
    for (double** p : {&b.ax, &b.ay, &b.az, &b.jx, &b.jy, &b.jz}) *p += at;
    hipLaunchKernelGGL((scf_jerk_kernel<S, LBV>), dim3(unsigned((b.n + 255) / 256)), dim3(256), lds, st, b);
  }
}

template <typename S>
int launch_jerk_lb(const JerkArgs& a, int grid, const JerkBatch* bi, hipStream_t st) {
  const int lb = a.lmax <= 2 ? 2 : (a.lmax + 1) / 2 * 2;
  switch (lb) {
    case 2: launch_jerk_kernel<S, 2>(a, grid, bi, st); break;
    case 4: launch_jerk_kernel<S, 4>(a, grid, bi, st); break;
    case 6: launch_jerk_kernel<S, 6>(a, grid, bi, st); break;
    case 8: launch_jerk_kernel<S, 8>(a, grid, bi, st); break;
    case 10: launch_jerk_kernel<S, 10>(a, grid, bi, st); break;
    case 12: launch_jerk_kernel<S, 12>(a, grid, bi, st); break;
    case 14: launch_jerk_kernel<S, 14>(a, grid, bi, st); break;
    default:
      set_error("internal: no jerk kernel bucket");
      return ETICS_EUNSUPPORTED;
  }
  return hip_fail(hipGetLastError(), "scf_jerk_kernel launch");
}

int launch_jerk_prep(const double* A, const double* B, const double* Ad, const double* Bd, int nmax,
                     int lmax, int nsys, int prec, void* cf, hipStream_t st) {
  if (prec != ETICS_FP64)
    return launch_force_prep_mm(A, B, Ad, Bd, nmax, lmax, nsys, kBasisHO, reinterpret_cast<float*>(cf), st);
  const int K = coeff_count(nmax, lmax);
  const int pb = int((int64_t(nsys) * K + 255) / 256);
  hipLaunchKernelGGL(scf_jerk_prep_kernel, dim3(pb), dim3(256), 0, st, A, B, Ad, Bd, nmax, lmax, nsys,
                     reinterpret_cast<Dual<double>*>(cf));
  return hip_fail(hipGetLastError(), "scf_jerk_prep_kernel launch");
}

int launch_jerk_any(const JerkArgs& a, int prec, int grid, const JerkBatch* bi, hipStream_t st) {
  return prec == ETICS_FP64 ? launch_jerk_lb<double>(a, grid, bi, st) : launch_jerk_lb<float>(a, grid, bi, st);
}

}  // namespace

int launch_scf_jerk(const double* x, const double* y, const double* z, const double* vx,
                    const double* vy, const double* vz, int64_t n, int nmax, int lmax,
                    const double* A, const double* B, const double* Ad, const double* Bd, int prec,
                    double* ax, double* ay, double* az, double* jx, double* jy, double* jz, void* ws,
                    hipStream_t st) {
  int rc = launch_jerk_prep(A, B, Ad, Bd, nmax, lmax, 1, prec, ws, st);
  if (rc || n == 0) return rc;
  JerkArgs a{};
  a.x = x;
  a.y = y;
  a.z = z;
  a.vx = vx;
  a.vy = vy;
  a.vz = vz;
  a.n = n;
  a.cf = ws;
  a.ax = ax;
  a.ay = ay;
  a.az = az;
  a.jx = jx;
  a.jy = jy;
  a.jz = jz;
  a.K = coeff_count(nmax, lmax);
  a.nmax = nmax;
  a.lmax = lmax;
  return launch_jerk_any(a, prec, 0, nullptr, st);
}

// ---------------------------------------------------------------- Hermite driver
namespace {

struct HermiteLayout {
  size_t off_ustart, off_usys, off_partials, off_prep, off_A, off_B, off_Ad, off_Bd, off_state, total;
  CoeffPlan plan;
  bool ok;
};

// workspace: unit tables, partial vectors (shared by both coefficient passes) and the
// prepared Dual coefficients (prep_region), A, B, dA/dt, dB/dt per system, and per particle a, j
// and the predicted position and velocity (12 doubles)
HermiteLayout hermite_layout(int64_t ntotal, int nsys, int nmax, int lmax, int prec) {
  HermiteLayout L{};
  L.ok = make_coeff_plan(ntotal, nmax, lmax, prec, &L.plan, kBasisHO, true);
  if (!L.ok) return L;
  const int K = coeff_count(nmax, lmax);
  const int mu = max_units(ntotal, nsys, L.plan.unit);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align_up(o + (bytes > 0 ? bytes : 1), 256);
    return at;
  };
  const size_t nn = size_t(ntotal > 0 ? ntotal : 1);
  L.off_ustart = take(size_t(nsys + 1) * 4);
  L.off_usys = take(size_t(mu) * 4);
  const PrepRegion r = prep_region(o, mu, nsys, K, size_t(8) * K, jerk_prep_bytes(nmax, lmax, prec), prec);
  L.off_partials = r.off_partials;
  L.off_prep = r.off_prep;
  o = r.end;
  L.off_A = take(size_t(nsys) * K * 8);
  L.off_B = take(size_t(nsys) * K * 8);
  L.off_Ad = take(size_t(nsys) * K * 8);
  L.off_Bd = take(size_t(nsys) * K * 8);
  L.off_state = take(12 * nn * 8);
  L.total = o;
  return L;
}

struct HermiteCall {
  double *x, *y, *z, *vx, *vy, *vz;
  const double* m;
  const int64_t* offsets;
  int nsys;
  int64_t ntotal;
  int nmax, lmax, prec;
  double dt;
  void* ws;
  size_t ws_bytes;
  int device;
  int plan[7];
};

bool same_call(const HermiteCall& a, const HermiteCall& b) {
  return a.x == b.x && a.y == b.y && a.z == b.z && a.vx == b.vx && a.vy == b.vy && a.vz == b.vz &&
         a.m == b.m && a.offsets == b.offsets && a.nsys == b.nsys && a.ntotal == b.ntotal &&
         a.nmax == b.nmax && a.lmax == b.lmax && a.prec == b.prec && a.dt == b.dt && a.ws == b.ws &&
         a.ws_bytes == b.ws_bytes && a.device == b.device && std::memcmp(a.plan, b.plan, sizeof a.plan) == 0;
}

// One jerk evaluation of every system: coefficients and their derivatives at the field
// points (fx.., fv..), reductions, rescale, then the jerk pass in `mode`.
int evaluate(const HermiteCall& c, const HermiteLayout& L, int mode, bool at_state, hipStream_t st) {
  char* base = reinterpret_cast<char*>(c.ws);
  const int* ustart = reinterpret_cast<const int*>(base + L.off_ustart);
  const int* usys = reinterpret_cast<const int*>(base + L.off_usys);
  double* A = reinterpret_cast<double*>(base + L.off_A);
  double* B = reinterpret_cast<double*>(base + L.off_B);
  double* Ad = reinterpret_cast<double*>(base + L.off_Ad);
  double* Bd = reinterpret_cast<double*>(base + L.off_Bd);
  double* s = reinterpret_cast<double*>(base + L.off_state);
  const int64_t n = c.ntotal;
  double *ax = s, *ay = s + n, *az = s + 2 * n, *jx = s + 3 * n, *jy = s + 4 * n, *jz = s + 5 * n;
  double *px = s + 6 * n, *py = s + 7 * n, *pz = s + 8 * n, *pvx = s + 9 * n, *pvy = s + 10 * n,
         *pvz = s + 11 * n;
  const double *fx = at_state ? c.x : px, *fy = at_state ? c.y : py, *fz = at_state ? c.z : pz;
  const double *fvx = at_state ? c.vx : pvx, *fvy = at_state ? c.vy : pvy, *fvz = at_state ? c.vz : pvz;
  const CoeffPlan& p = L.plan;
  int rc = launch_scf_coeffs_batched(p, fx, fy, fz, c.m, c.offsets, ustart, usys, c.nsys, n, A, B,
                                     base + L.off_partials, st);
  if (rc) return rc;
  rc = launch_scf_coeffs_dot_batched(p, fx, fy, fz, fvx, fvy, fvz, c.m, c.offsets, ustart, usys, c.nsys, n,
                                     Ad, Bd, base + L.off_partials, st);
  if (rc) return rc;
  rc = launch_jerk_prep(A, B, Ad, Bd, c.nmax, c.lmax, c.nsys, c.prec, base + L.off_prep, st);
  if (rc) return rc;
  JerkArgs a{};
  a.x = fx;
  a.y = fy;
  a.z = fz;
  a.vx = fvx;
  a.vy = fvy;
  a.vz = fvz;
  a.n = n;
  a.cf = base + L.off_prep;
  a.ax = ax;
  a.ay = ay;
  a.az = az;
  a.jx = jx;
  a.jy = jy;
  a.jz = jz;
  a.sx = c.x;
  a.sy = c.y;
  a.sz = c.z;
  a.svx = c.vx;
  a.svy = c.vy;
  a.svz = c.vz;
  a.px = px;
  a.py = py;
  a.pz = pz;
  a.pvx = pvx;
  a.pvy = pvy;
  a.pvz = pvz;
  a.K = coeff_count(c.nmax, c.lmax);
  a.nmax = c.nmax;
  a.lmax = c.lmax;
  a.mode = mode;
  a.dt = c.dt;
  const JerkBatch bi{c.offsets, ustart, usys, c.nsys, p.unit, p.split};
  return launch_jerk_any(a, c.prec, max_units(n, c.nsys, p.unit) * p.split, &bi, st);
}

struct GraphCache {
  bool valid = false;
  HermiteCall call{};
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipStream_t capture = nullptr;
};

std::mutex g_graph_mutex;
GraphCache g_graph;

void drop_graph(GraphCache& g) {
  if (g.exec) (void)hipGraphExecDestroy(g.exec);
  if (g.graph) (void)hipGraphDestroy(g.graph);
  g.exec = nullptr;
  g.graph = nullptr;
  g.valid = false;
}

}  // namespace

size_t hermite_ws_bytes(int64_t ntotal, int nsys, int nmax, int lmax, int prec) {
  const HermiteLayout L = hermite_layout(ntotal, nsys, nmax, lmax, prec);
  return L.ok ? L.total : 0;
}

int run_hermite(double* x, double* y, double* z, double* vx, double* vy, double* vz,
                const double* m, const int64_t* offsets, int nsys, int64_t ntotal, int nmax, int lmax,
                int prec, double dt, int nsteps, int flags, void* ws, size_t ws_bytes, hipStream_t st) {
  HermiteCall c{x, y, z, vx, vy, vz, m, offsets, nsys, ntotal, nmax, lmax, prec, dt, ws, ws_bytes, 0, {}};
  struct HookPause {
    bool prev;
    HookPause() : prev(timing_hook().suspended) { timing_hook().suspended = true; }
    ~HookPause() { timing_hook().suspended = prev; }
  } pause;
  int rc = hip_fail(hipGetDevice(&c.device), "hipGetDevice");
  if (rc) return rc;
  const HermiteLayout L = hermite_layout(ntotal, nsys, nmax, lmax, prec);
  if (!L.ok) {
    set_error("no tile plan for these cutoffs");
    return ETICS_EUNSUPPORTED;
  }
  if (ws_bytes < L.total) {
    set_error("workspace too small: need " + std::to_string(L.total) + " bytes");
    return ETICS_EWORKSPACE;
  }
  const CoeffPlan& plan = L.plan;
  const int shape[7] = {plan.nw, plan.tp, plan.streams, plan.grid_mult, plan.unit, plan.split, plan.mfma ? 2 : 1};
  std::memcpy(c.plan, shape, sizeof shape);
  char* base = reinterpret_cast<char*>(ws);
  rc = launch_units(offsets, nsys, ntotal, plan.unit, reinterpret_cast<int*>(base + L.off_ustart),
                    reinterpret_cast<int*>(base + L.off_usys), st);
  if (rc || nsteps < 1) return rc;
  // a, j at the starting state, and the first prediction
  rc = evaluate(c, L, kStart, true, st);
  if (rc) return rc;
  if ((flags & ETICS_LEAPFROG_EAGER) || nsteps == 1) {
    for (int k = 1; k < nsteps; ++k) {
      rc = evaluate(c, L, kStep, false, st);
      if (rc) return rc;
    }
    return evaluate(c, L, kLast, false, st);
  }
  std::lock_guard<std::mutex> lock(g_graph_mutex);
  if (!g_graph.valid || !same_call(g_graph.call, c)) {
    drop_graph(g_graph);
    if (!g_graph.capture) {
      rc = hip_fail(hipStreamCreateWithFlags(&g_graph.capture, hipStreamNonBlocking),
                    "hipStreamCreateWithFlags");
      if (rc) return rc;
    }
    rc = hip_fail(hipStreamBeginCapture(g_graph.capture, hipStreamCaptureModeThreadLocal),
                  "hipStreamBeginCapture");
    if (rc) return rc;
    const int rs = evaluate(c, L, kStep, false, g_graph.capture);
    hipGraph_t graph = nullptr;
    rc = hip_fail(hipStreamEndCapture(g_graph.capture, &graph), "hipStreamEndCapture");
    if (rs) {
      if (graph) (void)hipGraphDestroy(graph);
      return rs;
    }
    if (rc) return rc;
    g_graph.graph = graph;
    rc = hip_fail(hipGraphInstantiate(&g_graph.exec, graph, nullptr, nullptr, 0), "hipGraphInstantiate");
    if (rc) {
      drop_graph(g_graph);
      return rc;
    }
    g_graph.call = c;
    g_graph.valid = true;
  }
  for (int k = 1; k < nsteps; ++k) {
    rc = hip_fail(hipGraphLaunch(g_graph.exec, st), "hipGraphLaunch");
    if (rc) return rc;
  }
  return evaluate(c, L, kLast, false, st);
}

}  // namespace etics
