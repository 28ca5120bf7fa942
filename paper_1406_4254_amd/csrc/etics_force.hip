// etics_force.hip -- SCF potential and acceleration on gfx950 (MI355X).
//
// The second part of an SCF force calculation (paper Section 3.3): every particle's
// potential and acceleration from the coefficients A, B.  One particle per lane; the
// synthesis (radial recurrences and sums, angular synthesis, rotation to Cartesian
// components) is in etics_force_synth.hpp.  FP32 runs the radial sums on the matrix
// cores, FP64 as FMAs on coefficients broadcast from LDS.  In the batched leapfrog the
// epilogue applies the kicks (and drift) to the particle instead of storing its
// acceleration.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "etics_device.hpp"
#include "etics_force_synth.hpp"
#include "etics_internal.hpp"

namespace etics {

// ------------------------------------------------------------------ force prep
// Coefficients rescaled for the force kernel, in compute precision:
//   U, V: -sqrt(4pi) k_n (A, B)            (potential / radial part, with monic C_n)
//   W, X: -sqrt(4pi) 2 a_l c k'_{n-1} (A, B)  (d/dr part: dC_n^(a)/dxi = 2a C_{n-1}^(a+1))
// where dxi/dr = c g(r): Hernquist-Ostriker c = 2, g = u^2; Clutton-Brock c = 4,
// g = t u^3 (g is applied per particle by the force kernel).
// The scale of every (basis, n, l) is a constant (as loops of FP64 divisions in the kernel
// they were most of its 5 to 6 us).
struct ForceScales {
  double su[2][NCAP + 1][LCAP + 1], sw[2][NCAP + 1][LCAP + 1];
};
constexpr ForceScales make_force_scales() {
  ForceScales t{};
  constexpr double s4 = -2.0 * 0x1.c5bf891b4ef6ap+0;  // -sqrt(4 pi), rounded as sqrt(kPi)
  for (int b = 0; b < 2; ++b)
    for (int n = 0; n <= NCAP; ++n)
      for (int l = 0; l <= LCAP; ++l) {
        const double al = basis_alpha(b, l);
        const double dxi_c = b == kBasisCB ? 4.0 : 2.0;
        t.su[b][n][l] = s4 * gegen_k(n, al);
        t.sw[b][n][l] = n >= 1 ? s4 * 2.0 * al * dxi_c * gegen_k(n - 1, al + 1.0) : 0.0;
      }
  return t;
}
static __constant__ ForceScales g_force_scales = make_force_scales();

// FP64: two arrays of K, [0,K) U, [K,2K) V (RadialF64 derives the d/dr part)
__global__ __launch_bounds__(256) void scf_force_prep_kernel(const double* __restrict__ A,
                                                            const double* __restrict__ B,
                                                            int nmax, int lmax, int nsys, int basis,
                                                            double* __restrict__ cf) {
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
  const double su = g_force_scales.su[basis][n][l];
  const double a = A[g], b = B[g];
  double* c = cf + size_t(sys) * 2 * K;
  c[k] = su * a;
  c[K + k] = su * b;
}

// FP32: the quad layout of RadialMM, one value per thread and trip; with Ad, Bd (the jerk)
// each system's coefficients are followed by their time derivatives
__global__ __launch_bounds__(256) void scf_force_prep_mm_kernel(const double* __restrict__ A,
                                                               const double* __restrict__ B,
                                                               const double* __restrict__ Ad,
                                                               const double* __restrict__ Bd,
                                                               int nmax, int lmax, int nsys, int basis,
                                                               float* __restrict__ cf) {
  const int Q = mm_offset(lmax + 1, nmax);
  for (int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; g < int64_t(nsys) * Q;
       g += int64_t(gridDim.x) * blockDim.x) {
    const int sys = int(g / Q);
    int e = int(g - int64_t(sys) * Q);
    const int rep = 1 + 4 * mm_pairs(nmax);  // runs of padded slots per l
    int l = 0;
    while (e >= slot_pad(l, 4) * rep) {
      e -= slot_pad(l, 4) * rep;
      ++l;
    }
    const int P = slot_pad(l, 4);
    const int run = e / P, slot = e - run * P;
    // run 0: order 0 of U, V; then per pair j: U, V of 1+2j, of 2+2j, W, X of 1+2j, of 2+2j
    const int n = run == 0 ? 0 : 1 + 2 * ((run - 1) / 4) + ((run - 1) & 1);
    const bool deriv = run > 0 && (((run - 1) >> 1) & 1);
    float v = 0.f, d = 0.f;
    if (n <= nmax && slot <= 2 * l) {
      const int m = slot <= l ? slot : slot - l;
      const int K = (nmax + 1) * (lmax + 1) * (lmax + 2) / 2;
      const int64_t k = int64_t(sys) * K + n * ((lmax + 1) * (lmax + 2) / 2) + l * (l + 1) / 2 + m;
      const double scale = deriv ? g_force_scales.sw[basis][n][l] : g_force_scales.su[basis][n][l];
      v = float(scale * (slot <= l ? A[k] : B[k]));
      if (Ad) d = float(scale * (slot <= l ? Ad[k] : Bd[k]));
    }
    float* const c = cf + size_t(sys) * (Ad ? 2 * Q : Q);
    c[g - int64_t(sys) * Q] = v;
    if (Ad) c[Q + (g - int64_t(sys) * Q)] = d;
  }
}

// ------------------------------------------------------------------------ force
struct ForceArgs {
  const double *x, *y, *z;
  int64_t n;
  const void* cf;  // prepared coefficients: quad layout (FP32) or 2K (FP64)
  double *pot, *ax, *ay, *az;
  int K, nmax, lmax;
  int want_pot;
  LfUpdate lf;     // lf.mode = 0: write a; otherwise update v (and x) instead
};

// the outputs of point i: potential and acceleration, or the leapfrog update
template <typename T, bool ACC>
__device__ __forceinline__ void force_store(const ForceArgs& a, int64_t i, T pot, T gx, T gy, T gz) {
  if (a.want_pot) a.pot[i] = double(pot);
  if constexpr (ACC) {
    if (a.lf.mode == 0) {
      a.ax[i] = double(gx);
      a.ay[i] = double(gy);
      a.az[i] = double(gz);
    } else {
      // leapfrog: closing kick, then (mode 2) the next step's opening kick and drift;
      // only this thread touches particle i, so x is updated in place after its use
      const double h = a.lf.h;
      double vx = __builtin_fma(h, double(gx), a.lf.vx[i]);
      double vy = __builtin_fma(h, double(gy), a.lf.vy[i]);
      double vz = __builtin_fma(h, double(gz), a.lf.vz[i]);
      if (a.lf.mode == 2) {
        vx = __builtin_fma(h, double(gx), vx);
        vy = __builtin_fma(h, double(gy), vy);
        vz = __builtin_fma(h, double(gz), vz);
        a.lf.x[i] = __builtin_fma(a.lf.dt, vx, a.x[i]);
        a.lf.y[i] = __builtin_fma(a.lf.dt, vy, a.y[i]);
        a.lf.z[i] = __builtin_fma(a.lf.dt, vz, a.z[i]);
      }
      a.lf.vx[i] = vx;
      a.lf.vy[i] = vy;
      a.lf.vz[i] = vz;
    }
  }
}

// FP32: potential / acceleration of the points [i0, i1), one per lane, from one system's
// prepared coefficients.  The matrix cores need every lane of a wavefront, so the loop
// is uniform over the workgroup and a lane past the end computes a point at the origin.
// NEXT: the coordinates of a lane's next point are loaded with what the leapfrog update
// of the current one needs, after the synthesis (one wait instead of two; at lmax > 6
// the registers for it are not there: 93 -> 143 us at N = 10^6, (10, 10)).
template <int LB, bool ACC, int BASIS, bool NEXT>
__device__ __forceinline__ void force_points_mm(const ForceArgs& a, const float* cf, int64_t i0, int64_t i1,
                                                int64_t stride) {
  RadialMM<float, ACC, BASIS> rad(cf, a.nmax, a.lmax);
  double x = 0.0, y = 0.0, z = 0.0;
  auto load = [&](int64_t i) {
    const bool valid = i < i1;
    x = valid ? a.x[i] : 0.0;
    y = valid ? a.y[i] : 0.0;
    z = valid ? a.z[i] : 0.0;
  };
  if constexpr (NEXT) load(i0 + threadIdx.x);
  rad.template start<0>();
  for (; i0 < i1; i0 += stride) {
    const int64_t i = i0 + threadIdx.x;
    if constexpr (!NEXT) load(i);
    const Sph<float> s = sph<float, BASIS, true>(x, y, z);
    const ForceOut<float> o = synth_point<float, LB, ACC, BASIS>(s, rad, a.lmax);
    if constexpr (NEXT) load(i + stride);
    // before the stores: loads and stores are waited for in order
    rad.template start<0>();
    if (i < i1) force_store<float, ACC>(a, i, o.pot, o.gx, o.gy, o.gz);
  }
}

template <typename T, int LB, bool ACC, int BASIS>
__global__ __launch_bounds__(256, LB <= 10 ? 4 : 3) void scf_force_kernel(const ForceArgs a) {
  static_assert(sizeof(T) == 4, "FP64 runs scf_force_f64_kernel");
  force_points_mm<LB, ACC, BASIS, false>(a, reinterpret_cast<const float*>(a.cf), int64_t(blockIdx.x) * blockDim.x,
                                         a.n, int64_t(gridDim.x) * blockDim.x);
}

// FP64.  One point per lane and no loop over points: in a loop the compiler hoists the
// FP64 constants (an SGPR pair each) out of it and spills them to vector lanes, 640 lane
// moves per point at (10, 10).  LDS: the workgroup copies the prepared coefficients to
// LDS first, as [K][2], and every lane reads them as broadcast VGPR operands.  Such reads
// are what bounds the pass (a 16-byte broadcast takes the LDS 8 cycles for 64 lanes,
// whatever it feeds): two doubles per coefficient instead of four, each feeding two FMAs,
// took N = 10^6, (10, 10) from 261 to 197 us a call and N = 5 10^5, (20, 14) from 783 to
// 333 us.  Otherwise (potential only, where a read feeds one FMA per double) the
// coefficients are scalar operands: 119 -> 96 us at N = 10^6, (10, 10).
template <bool ACC, int BASIS, int LB, typename Radial>
__device__ __forceinline__ void force_point_f64(const ForceArgs& a, Radial rad, int64_t i) {
  const Sph<double> s = sph<double, BASIS, true>(a.x[i], a.y[i], a.z[i]);
  const ForceOut<double> o = synth_point<double, LB, ACC, BASIS>(s, rad, a.lmax);
  force_store<double, ACC>(a, i, o.pot, o.gx, o.gy, o.gz);
}
// cf [2][K] to the workgroup's LDS [K][2]
__device__ __forceinline__ void coeffs_to_lds(const double* cf, int K, double* lds) {
  for (int k = threadIdx.x; k < 2 * K; k += blockDim.x) {
    const int which = k >= K;
    lds[2 * (k - which * K) + which] = cf[k];
  }
  __syncthreads();
}
template <int LB, bool ACC, int BASIS, bool LDS>
__global__ __launch_bounds__(256, 2) void scf_force_f64_kernel(const ForceArgs a) {
  extern __shared__ __align__(16) double lds_cf[];
  const double* cf = reinterpret_cast<const double*>(a.cf);
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if constexpr (LDS) {
    coeffs_to_lds(cf, a.K, lds_cf);
    if (i >= a.n) return;
    force_point_f64<ACC, BASIS, LB>(
        a, RadialF64<ACC, BASIS, LdsPtr<double>, true>{(LdsPtr<double>)(lds_cf), a.K, a.nmax, a.lmax}, i);
  } else {
    if (i >= a.n) return;
    force_point_f64<ACC, BASIS, LB>(
        a, RadialF64<ACC, BASIS, ConstPtr<double>, false>{(ConstPtr<double>)(cf), a.K, a.nmax, a.lmax}, i);
  }
}

// batched systems: `split` workgroups per unit of `unit` particles of one system (each a
// contiguous part of it), so the coefficients are uniform across the workgroup; splitting
// the coefficient kernel's units gives the force pass more workgroups.  FP64: the
// system's prepared coefficients are copied to LDS as [K][2] first, as in
// scf_force_f64_kernel; FP32: as in scf_force_kernel.
// The potential alone at lmax > 10 in FP64 asks for one wavefront a SIMD: held to the registers
// of two, the compiler keeps fewer LDS reads in flight.  Two / one, us a call: 128 systems (9, 12)
// 286 / 248, (20, 14) 780 / 676; 16 systems of 1000 (9, 12) 90 / 72, (20, 14) 243 / 195.
template <typename T, int LB, bool ACC>
__global__ __launch_bounds__(256, sizeof(T) == 8 ? (LB <= 6 ? 3 : LB > 10 && !ACC ? 1 : 2) : LB <= 10 ? 4 : 3) void scf_force_batched_kernel(const ForceArgs a,
                                                                const int64_t* __restrict__ offsets,
                                                                const int* __restrict__ ustart,
                                                                const int* __restrict__ usys,
                                                                int nsys, int unit, int split) {
  extern __shared__ __align__(16) double lds_cf[];
  const int u = blockIdx.x / split;
  const int part = blockIdx.x % split;
  if (u >= ustart[nsys]) return;
  const int sys = usys[u];
  int64_t b = offsets[sys], e = offsets[sys + 1];
  b = b < 0 ? 0 : (b > a.n ? a.n : b);
  e = e < b ? b : (e > a.n ? a.n : e);
  const int64_t kPart = (unit + split - 1) / split;
  const int64_t u0 = b + int64_t(u - ustart[sys]) * unit;
  const int64_t ue0 = u0 + unit < e ? u0 + unit : e;
  const int64_t ub = u0 + part * kPart < ue0 ? u0 + part * kPart : ue0;
  const int64_t ue = ub + kPart < ue0 ? ub + kPart : ue0;
  if (ub >= ue) return;
  if constexpr (sizeof(T) == 4) {
    const float* cf = reinterpret_cast<const float*>(a.cf) +
                      size_t(__builtin_amdgcn_readfirstlane(sys)) * mm_offset(a.lmax + 1, a.nmax);
    force_points_mm<LB, ACC, kBasisHO, LB <= 6>(a, cf, ub, ue, blockDim.x);
  } else {
    coeffs_to_lds(reinterpret_cast<const double*>(a.cf) + size_t(sys) * 2 * a.K, a.K, lds_cf);
    const RadialF64<ACC, kBasisHO, LdsPtr<double>, true> rad{(LdsPtr<double>)(lds_cf), a.K, a.nmax, a.lmax};
    for (int64_t i = ub + threadIdx.x; i < ue; i += blockDim.x) force_point_f64<ACC, kBasisHO, LB>(a, rad, i);
  }
}

int launch_force_prep_mm(const double* A, const double* B, const double* Ad, const double* Bd, int nmax, int lmax,
                         int nsys, int basis, float* cf, hipStream_t st) {
  // (many systems' values would be 2^32 threads, more than a grid holds)
  const int64_t values = int64_t(nsys) * mm_offset(lmax + 1, nmax), blocks = (values + 255) / 256;
  hipLaunchKernelGGL(scf_force_prep_mm_kernel, dim3(unsigned(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st, A, B,
                     Ad, Bd, nmax, lmax, nsys, basis, cf);
  return hip_fail(hipGetLastError(), "scf_force_prep_mm_kernel launch");
}

size_t force_prep_bytes(int nmax, int lmax, int prec) {
  return prec == ETICS_FP64 ? size_t(2) * coeff_count(nmax, lmax) * 8 : size_t(mm_offset(lmax + 1, nmax)) * 4;
}

namespace {

struct BatchInfo {
  const int64_t* offsets;
  const int* ustart;
  const int* usys;
  int nsys, unit, split;
};

// FP64, one point per lane.  Potential only: scalar coefficient operands for many points
// and lmax > 6, where the LDS reads bound the pass; elsewhere the scalar loads' latency
// shows.  LDS against scalar operands, us a call: (10, 10) 26 / 33 at 10^5 points, 43 / 45
// at 2 10^5, 60 / 59 at 4 10^5, 118 / 102 at 10^6; (10, 6) 25 / 30 at 4 10^5.
constexpr int64_t kScalarPoints = 400000;
template <bool ACC, int LBV, int BASIS>
void launch_force_f64(const ForceArgs& a, hipStream_t st) {
  const size_t lds = size_t(2) * a.K * sizeof(double);  // at most 40 KiB
  const bool scalar = !ACC && LBV > 6 && a.n >= kScalarPoints;
  // a grid holds less than 2^32 threads
  constexpr int64_t kMost = int64_t(1) << 30;
  for (int64_t at = 0; at < a.n; at += kMost) {
    ForceArgs b = a;
    b.n = a.n - at < kMost ? a.n - at : kMost;
    b.x += at;
    b.y += at;
    b.z += at;
    if (at > 0) {
      if (b.pot) b.pot += at;
      if (b.ax) b.ax += at;
      if (b.ay) b.ay += at;
      if (b.az) b.az += at;
    }
    const dim3 grid(unsigned((b.n + 255) / 256));
    if constexpr (!ACC && LBV > 6) {
      if (scalar) {
        hipLaunchKernelGGL((scf_force_f64_kernel<LBV, ACC, BASIS, false>), grid, dim3(256), 0, st, b);
        continue;
      }
    }
    hipLaunchKernelGGL((scf_force_f64_kernel<LBV, ACC, BASIS, true>), grid, dim3(256), lds, st, b);
  }
}

template <typename T, bool ACC, int LBV>
void launch_force_kernel(const ForceArgs& a, int basis, int grid, const BatchInfo* bi,
                         hipStream_t st) {
  if (bi) {
    const size_t lds = sizeof(T) == 8 ? size_t(2) * a.K * sizeof(T) : 0;
    hipLaunchKernelGGL((scf_force_batched_kernel<T, LBV, ACC>), dim3(grid), dim3(256), lds, st, a,
                       bi->offsets, bi->ustart, bi->usys, bi->nsys, bi->unit, bi->split);
  } else if constexpr (sizeof(T) == 8) {
    if (basis == kBasisCB)
      launch_force_f64<ACC, LBV, kBasisCB>(a, st);
    else
      launch_force_f64<ACC, LBV, kBasisHO>(a, st);
  } else if (basis == kBasisCB)
    hipLaunchKernelGGL((scf_force_kernel<T, LBV, ACC, kBasisCB>), dim3(grid), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((scf_force_kernel<T, LBV, ACC, kBasisHO>), dim3(grid), dim3(256), 0, st, a);
}

template <typename T, bool ACC>
int launch_force_lb(int lb, const ForceArgs& a, int basis, int grid, const BatchInfo* bi,
                    hipStream_t st) {
  switch (lb) {
    case 2: launch_force_kernel<T, ACC, 2>(a, basis, grid, bi, st); break;
    case 4: launch_force_kernel<T, ACC, 4>(a, basis, grid, bi, st); break;
    case 6: launch_force_kernel<T, ACC, 6>(a, basis, grid, bi, st); break;
    case 8: launch_force_kernel<T, ACC, 8>(a, basis, grid, bi, st); break;
    case 10: launch_force_kernel<T, ACC, 10>(a, basis, grid, bi, st); break;
    case 12: launch_force_kernel<T, ACC, 12>(a, basis, grid, bi, st); break;
    case 14: launch_force_kernel<T, ACC, 14>(a, basis, grid, bi, st); break;
    default:
      set_error("internal: no force kernel bucket");
      return ETICS_EUNSUPPORTED;
  }
  return hip_fail(hipGetLastError(), "scf_force_kernel launch");
}

int launch_prep(const double* A, const double* B, int nmax, int lmax, int nsys, int prec, int basis,
                void* ws, hipStream_t st) {
  if (prec != ETICS_FP64)
    return launch_force_prep_mm(A, B, nullptr, nullptr, nmax, lmax, nsys, basis, reinterpret_cast<float*>(ws), st);
  const int pb = int((int64_t(nsys) * coeff_count(nmax, lmax) + 255) / 256);
  hipLaunchKernelGGL(scf_force_prep_kernel, dim3(pb), dim3(256), 0, st, A, B, nmax, lmax, nsys, basis,
                     reinterpret_cast<double*>(ws));
  return hip_fail(hipGetLastError(), "scf_force_prep_kernel launch");
}

int launch_force_any(const ForceArgs& a, int prec, int outputs, int basis, int grid,
                     const BatchInfo* bi, hipStream_t st) {
  const int lb = a.lmax <= 2 ? 2 : (a.lmax + 1) / 2 * 2;
  const bool acc = (outputs & ETICS_ACC) != 0;
  int rc = hook_before(st);
  if (rc) return rc;
  if (prec == ETICS_FP64)
    rc = acc ? launch_force_lb<double, true>(lb, a, basis, grid, bi, st)
             : launch_force_lb<double, false>(lb, a, basis, grid, bi, st);
  else
    rc = acc ? launch_force_lb<float, true>(lb, a, basis, grid, bi, st)
             : launch_force_lb<float, false>(lb, a, basis, grid, bi, st);
  return rc ? rc : hook_after(st);
}

ForceArgs make_force_args(const double* x, const double* y, const double* z, int64_t n, int nmax,
                          int lmax, int outputs, double* pot, double* ax, double* ay, double* az,
                          const void* cf) {
  ForceArgs a{};
  a.x = x;
  a.y = y;
  a.z = z;
  a.n = n;
  a.cf = cf;
  a.pot = pot;
  a.ax = ax;
  a.ay = ay;
  a.az = az;
  a.K = coeff_count(nmax, lmax);
  a.nmax = nmax;
  a.lmax = lmax;
  a.want_pot = (outputs & ETICS_POT) ? 1 : 0;
  return a;
}

}  // namespace

int launch_scf_force(const double* x, const double* y, const double* z, int64_t n, int nmax,
                     int lmax, const double* A, const double* B, int prec, int outputs,
                     double* pot, double* ax, double* ay, double* az, void* ws, hipStream_t st,
                     int basis) {
  int rc = launch_prep(A, B, nmax, lmax, 1, prec, basis, ws, st);
  if (rc || n == 0) return rc;
  const ForceArgs a = make_force_args(x, y, z, n, nmax, lmax, outputs, pot, ax, ay, az, ws);
  int64_t grid = (n + 255) / 256;
  if (grid > 65536) grid = 65536;
  return launch_force_any(a, prec, outputs, basis, int(grid), nullptr, st);
}

int launch_scf_force_batched(const CoeffPlan& plan, const double* x, const double* y,
                             const double* z, const int64_t* offsets, const int* ustart,
                             const int* usys, int nsys, int64_t ntotal, const double* A,
                             const double* B, int outputs, double* pot, double* ax, double* ay,
                             double* az, void* prep, hipStream_t st, const LfUpdate* lf) {
  const int nmax = plan.nmax, lmax = plan.lmax, prec = plan.prec;
  int rc = launch_prep(A, B, nmax, lmax, nsys, prec, kBasisHO, prep, st);
  if (rc || ntotal == 0) return rc;
  ForceArgs a = make_force_args(x, y, z, ntotal, nmax, lmax, outputs, pot, ax, ay, az, prep);
  if (lf) a.lf = *lf;
  const BatchInfo bi{offsets, ustart, usys, nsys, plan.unit, plan.split};
  return launch_force_any(a, prec, outputs, kBasisHO, max_units(ntotal, nsys, plan.unit) * plan.split,
                          &bi, st);
}

}  // namespace etics
