// etics_direct.hip -- unsoftened direct-summation potential and acceleration (FP64).
//
// The accuracy study of the paper (Section 4.1) compares the expansion forces with
// direct summation, in double precision and without softening, and with the smooth
// force of the model.  For every particle i:
//   Phi_i = -sum_{j, r_ij > 0} m_j / r_ij,   a_i = sum_{j, r_ij > 0} m_j (x_j - x_i) / r_ij^3
// (G = 1).  The particle itself, and any other particle at exactly the same position,
// adds nothing.
//
// What bounds it is FP64 issue: 23 instructions in about 26 issue slots a pair (0.83 of the
// slots taken), of which the reciprocal square root took most when it came from the math
// library (49 slots a pair; 12.1 ms at n = 10^5, now 8.7 to 9.6 from run to run; n = 1000:
// 70 -> 11 us).  The sources are split over the lanes and wavefronts of a workgroup, so
// that small n fills the chip too and large n leaves no long last round:
// a workgroup holds 16 NT targets (16 lanes, NT targets a lane), its 4 WAVES slices of
// lanes each take every (4 WAVES)-th source, and the slices are added in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "etics_device.hpp"
#include "etics_internal.hpp"

namespace etics {

constexpr int kTargetLanes = 16;

// 1 / sqrt(r2) for a positive finite r2, else 0 (no distance, or one whose square
// overflows, adds nothing): the hardware estimate (about 2^-23) and one step of third
// order, y (1 + e/2 + 3 e^2 / 8) with e = 1 - r2 y^2, which leaves the last rounding.
__device__ __forceinline__ double pair_rinv(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double e = fma_(-(r2 * y), y, 1.0);
  const double z = fma_(y * e, fma_(0.375, e, 0.5), y);
  return __builtin_amdgcn_class(r2, 0x180) ? z : 0.0;  // positive normal or subnormal
}

template <int NT, int WAVES, bool POT, bool ACC>
__global__ __launch_bounds__(64 * WAVES) void direct_force_kernel(
    const double* __restrict__ x, const double* __restrict__ y, const double* __restrict__ z,
    const double* __restrict__ m, int64_t n, double* __restrict__ pot, double* __restrict__ ax,
    double* __restrict__ ay, double* __restrict__ az) {
  constexpr int kSlices = 4 * WAVES;
  constexpr int NV = (POT ? 1 : 0) + (ACC ? 3 : 0);
  __shared__ double sums[NV][kSlices][NT * kTargetLanes];
  const int64_t group = int64_t(blockIdx.y) * gridDim.x + blockIdx.x;
  if (group * (NT * kTargetLanes) >= n) return;
  const int tl = threadIdx.x % kTargetLanes, slice = threadIdx.x / kTargetLanes;
  const int64_t t0 = group * (NT * kTargetLanes) + tl;
  double px[NT], py[NT], pz[NT], P[NT] = {}, gx[NT] = {}, gy[NT] = {}, gz[NT] = {};
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const int64_t i = t0 + k * kTargetLanes;
    px[k] = i < n ? x[i] : 0.0;
    py[k] = i < n ? y[i] : 0.0;
    pz[k] = i < n ? z[i] : 0.0;
  }
  auto add = [&](double sx, double sy, double sz, double sm) {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const double dx = sx - px[k], dy = sy - py[k], dz = sz - pz[k];
      const double rinv = pair_rinv(dx * dx + dy * dy + dz * dz);
      const double mr = sm * rinv;
      if constexpr (POT) P[k] -= mr;
      if constexpr (ACC) {
        const double mr3 = mr * rinv * rinv;
        gx[k] += mr3 * dx;
        gy[k] += mr3 * dy;
        gz[k] += mr3 * dz;
      }
    }
  };
  int64_t j = slice;
  constexpr int U = 4;  // sources of a trip, loaded together
  for (; j + (U - 1) * kSlices < n; j += U * kSlices) {
    double sx[U], sy[U], sz[U], sm[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sx[u] = x[j + u * kSlices];
      sy[u] = y[j + u * kSlices];
      sz[u] = z[j + u * kSlices];
      sm[u] = m[j + u * kSlices];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) add(sx[u], sy[u], sz[u], sm[u]);
  }
  for (; j < n; j += kSlices) add(x[j], y[j], z[j], m[j]);

#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const int e = k * kTargetLanes + tl;
    if constexpr (POT) sums[0][slice][e] = P[k];
    if constexpr (ACC) {
      sums[NV - 3][slice][e] = gx[k];
      sums[NV - 2][slice][e] = gy[k];
      sums[NV - 1][slice][e] = gz[k];
    }
  }
  __syncthreads();
  for (int o = threadIdx.x; o < NV * NT * kTargetLanes; o += 64 * WAVES) {
    const int v = o / (NT * kTargetLanes), e = o % (NT * kTargetLanes);
    const int64_t i = group * (NT * kTargetLanes) + e;
    if (i >= n) continue;
    double s = sums[v][0][e];
    for (int q = 1; q < kSlices; ++q) s += sums[v][q][e];
    double* const out = POT && v == 0 ? pot : v == NV - 3 ? ax : v == NV - 2 ? ay : az;
    out[i] = s;
  }
}

namespace {
template <int NT, int WAVES>
void launch_direct(const double* x, const double* y, const double* z, const double* m, int64_t n,
                   int outputs, double* pot, double* ax, double* ay, double* az, hipStream_t st) {
  // rows of workgroups: a row holds less than 2^32 threads (one row of all n < 2^31 targets would not)
  const int64_t groups = (n + NT * kTargetLanes - 1) / (NT * kTargetLanes);
  const int64_t row = groups < 4096 ? groups : 4096;
  const dim3 grid(unsigned(row), unsigned((groups + row - 1) / row)), block(64 * WAVES);
  if (outputs == ETICS_POT)
    hipLaunchKernelGGL((direct_force_kernel<NT, WAVES, true, false>), grid, block, 0, st, x, y, z, m, n, pot, ax, ay, az);
  else if (outputs == ETICS_ACC)
    hipLaunchKernelGGL((direct_force_kernel<NT, WAVES, false, true>), grid, block, 0, st, x, y, z, m, n, pot, ax, ay, az);
  else
    hipLaunchKernelGGL((direct_force_kernel<NT, WAVES, true, true>), grid, block, 0, st, x, y, z, m, n, pot, ax, ay, az);
}
}  // namespace

int launch_direct_force(const double* x, const double* y, const double* z, const double* m,
                        int64_t n, int outputs, double* pot, double* ax, double* ay, double* az,
                        hipStream_t st) {
  int rc = hook_before(st);
  if (rc) return rc;
  // Targets a lane: the fewest rounds of workgroups over the 256 CUs, each round as long
  // as its targets times what a pair costs.  The source reads (four loads for NT pairs a
  // lane) weigh on small NT: us a call with 1, 2, 3, 4, 8 targets a lane 211, 143, 107,
  // 124, 281 at n = 10^4 and 16900, 9300, 8700, 8700, 10000 at 10^5.
  constexpr int kPairCost[4] = {19, 11, 10, 10};
  int nt = 1;
  int64_t best = 0;
  for (int k = 1; k <= 4; ++k) {
    const int64_t groups = (n + k * kTargetLanes - 1) / (k * kTargetLanes);
    const int64_t cost = (groups + 255) / 256 * k * kPairCost[k - 1];
    if (k == 1 || cost < best) {
      best = cost;
      nt = k;
    }
  }
  switch (nt) {
    case 1: launch_direct<1, 4>(x, y, z, m, n, outputs, pot, ax, ay, az, st); break;
    case 2: launch_direct<2, 4>(x, y, z, m, n, outputs, pot, ax, ay, az, st); break;
    case 3: launch_direct<3, 4>(x, y, z, m, n, outputs, pot, ax, ay, az, st); break;
    default: launch_direct<4, 8>(x, y, z, m, n, outputs, pot, ax, ay, az, st); break;
  }
  rc = hip_fail(hipGetLastError(), "direct_force_kernel launch");
  return rc ? rc : hook_after(st);
}

}  // namespace etics
