// etics_force_synth.hpp -- the per-point synthesis of the SCF potential and
// acceleration from prepared coefficients, shared by the force kernels
// (etics_force.hip) and the jerk kernels (etics_jerk.hip).
//
// For each l the two radial recurrences (Gegenbauer in monic form, for the potential
// and for d/dr) run over n, and the sums over n of recurrence value times coefficient
// (the same coefficient for every point) come from one of three sources: the matrix cores
// (RadialMM, FP32 and its Dual), or FMAs on coefficients read as uniform operands
// (RadialF64; RadialDual, FP64 with derivatives).  The l and m loops are compile-time, so
// the recurrence and derivative constants are instruction literals.  The angular synthesis
// uses division-free identities for dYbar/dtheta and m Ybar/sin(theta), and the result is
// rotated to Cartesian components.
// The compute type may carry time derivatives (Dual), which turns the same code into the
// jerk.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "etics_device.hpp"
#include "etics_internal.hpp"

namespace etics {

static __constant__ BasisTables<double> g_tab64 = make_tables<double>();

// A prepared coefficient read through the constant address space (wave-uniform, so a
// scalar load into SGPR operands); a Dual one member by member
template <typename T>
__device__ __forceinline__ T cload(const __attribute__((address_space(4))) T* p) {
  return *p;
}
template <typename S>
__device__ __forceinline__ Dual<S> cload(const __attribute__((address_space(4))) Dual<S>* p) {
  return Dual<S>(p->v, p->d);
}
// ... or from a workgroup's copy in LDS: every lane reads the same address (a broadcast)
// into VGPR operands (FP64 and Dual, where each coefficient would take two SGPRs)
template <typename T>
__device__ __forceinline__ T cload(const __attribute__((address_space(3))) T* p) {
  return *p;
}
template <typename S>
__device__ __forceinline__ Dual<S> cload(const __attribute__((address_space(3))) Dual<S>* p) {
  return Dual<S>(p->v, p->d);
}
template <typename T>
using ConstPtr = const __attribute__((address_space(4))) T*;
template <typename T>
using LdsPtr = const __attribute__((address_space(3))) T*;

// Potential and acceleration (-grad Phi, Cartesian) at a point with spherical
// coordinates s, from one system's prepared coefficients cf.  T is the compute type,
// or Dual<S> to carry every quantity's time derivative along the motion (the jerk).
template <typename T>
struct ForceOut {
  T pot, gx, gy, gz;
};

// Radial sums of one l over n, for every m: U, V (potential; cos and sin coefficients)
// from Chat_n and W, X (d/dr) from Ehat_{n-1} (parameter a_l + 1).  Order 0 is taken in
// closed form (Chat_0 = 1; it adds nothing to W, X since Ehat_{-1} = 0).
//
// RadialDual: FP64 with derivatives (Hernquist-Ostriker), one Dual FMA per coefficient.  The
// coefficients' four arrays are read through the constant address space (ConstPtr;
// wave-uniform scalar loads into SGPR operands), laid out [4][K], or in LDS (LdsPtr), with
// QUAD [K][4] (the four values of a coefficient side by side, two 16-byte reads each).
template <typename P, bool QUAD>
struct RadialDual {
  using T = Dual<double>;
  P cf;
  int K, nmax, lmax;

  template <int l>
  __device__ __forceinline__ void start() {}

  template <int l>
  __device__ __forceinline__ void sums(T xi, T (&U)[l + 1], T (&V)[l + 1], T (&W)[l + 1], T (&X)[l + 1]) {
    const int WK = QUAD ? 1 : K;      // offset from one array to the next
    constexpr int IS = QUAD ? 4 : 1;  // offset from one coefficient to the next
    const int L2 = (lmax + 1) * (lmax + 2) / 2;
    const P cfl = cf + l * (l + 1) / 2 * IS;
#pragma unroll
    for (int m = 0; m <= l; ++m) {
      U[m] = cload(cfl + m * IS);
      V[m] = m > 0 ? cload(cfl + WK + m * IS) : T(0);
      W[m] = T(0);
      X[m] = T(0);
    }
    T c2 = T(0), c1 = T(1);  // Chat_{n-2}, Chat_{n-1} for n = 1 (Chat_{-1} enters times 0)
    T e2 = T(0), e1 = T(1);  // Ehat_{n-2}, Ehat_{n-1} (parameter a_l + 1)
    const double* ql = g_tab64.q[l];
    const double* qdl = g_tab64.qd[l];
    // one order per trip keeps the coefficients of a trip in registers
    for (int nn = 1; nn <= nmax; ++nn) {
      const T c = recur(xi, c1, ql[nn], c2);  // Chat_nn
      const auto* cn = cfl + nn * L2 * IS;
#pragma unroll
      for (int m = 0; m <= l; ++m) {
        U[m] = fma_(c, cload(cn + m * IS), U[m]);
        if (m > 0) V[m] = fma_(c, cload(cn + WK + m * IS), V[m]);
      }
      c2 = c1;
      c1 = c;
#pragma unroll
      for (int m = 0; m <= l; ++m) {
        W[m] = fma_(e1, cload(cn + 2 * WK + m * IS), W[m]);
        if (m > 0) X[m] = fma_(e1, cload(cn + 3 * WK + m * IS), X[m]);
      }
      const T e = recur(xi, e1, qdl[nn], e2);  // Ehat_nn
      e2 = e1;
      e1 = e;
    }
  }
};

// RadialF64: plain FP64.  The d/dr family needs no coefficients of its own: with monic
// polynomials d Chat_n / d xi = n Ehat_{n-1}, so W, X take n c Ehat_{n-1} (dxi/dr = c g)
// times the coefficients of U, V, and every coefficient read feeds two FMAs.
template <bool ACC, int BASIS, typename P, bool PAIR>
struct RadialF64 {
  P cf;  // [2][K], or with PAIR [K][2]
  int K, nmax, lmax;

  template <int l>
  __device__ __forceinline__ void start() {}

  template <int l>
  __device__ __forceinline__ void sums(double xi, double (&U)[l + 1], double (&V)[l + 1], double (&W)[l + 1],
                                       double (&X)[l + 1]) {
    const int VK = PAIR ? 1 : K;
    constexpr int IS = PAIR ? 2 : 1;
    const BasisTables<double>& tb = g_tab64;
    const int L2 = (lmax + 1) * (lmax + 2) / 2;
    const P cfl = cf + l * (l + 1) / 2 * IS;
#pragma unroll
    for (int m = 0; m <= l; ++m) {
      U[m] = cload(cfl + m * IS);
      V[m] = m > 0 ? cload(cfl + VK + m * IS) : 0.0;
      W[m] = 0.0;
      X[m] = 0.0;
    }
    double c2 = 0.0, c1 = 1.0;  // Chat_{n-2}, Chat_{n-1} for n = 1
    double e2 = 0.0, e1 = 1.0;  // Ehat_{n-2}, Ehat_{n-1}
    double cn = 0.0;            // c n
    const double* ql = BASIS == kBasisCB ? tb.qcb[l] : tb.q[l];
    const double* qdl = BASIS == kBasisCB ? tb.qdcb[l] : tb.qd[l];
    auto step = [&](int nn, double& cA, double& cB, double& eA, double& eB) {
      cA = recur(xi, cB, ql[nn], cA);
      double ec = 0.0;
      if constexpr (ACC) {
        cn += BASIS == kBasisCB ? 4.0 : 2.0;
        ec = cn * eB;
      }
      const auto* p = cfl + nn * L2 * IS;
#pragma unroll
      for (int m = 0; m <= l; ++m) {
        const double a = cload(p + m * IS);
        U[m] = fma_(cA, a, U[m]);
        if constexpr (ACC) W[m] = fma_(ec, a, W[m]);
        if (m > 0) {
          const double b = cload(p + VK + m * IS);
          V[m] = fma_(cA, b, V[m]);
          if constexpr (ACC) X[m] = fma_(ec, b, X[m]);
        }
      }
      if constexpr (ACC) eA = recur(xi, eB, qdl[nn], eA);
    };
    int nn = 1;
    for (; nn + 1 <= nmax; nn += 2) {
      step(nn, c2, c1, e2, e1);
      step(nn + 1, c1, c2, e1, e2);
    }
    if (nn <= nmax) step(nn, c2, c1, e2, e1);
  }
};

// RadialMM: the sums on the matrix cores (FP32).  v_mfma_f32_4x4x1 multiplies, in each
// of 16 blocks, 4 A values (lanes 4b .. 4b+3) with 4 B values (the same lanes) into a
// 4 x 4 accumulator whose column j is the four registers of lane 4b+j.  With A = the
// coefficients of 4 (cos or sin) slots and B = the lane's own recurrence value, a lane
// so accumulates 4 slots of its own point: no lane moves, and each accumulator goes
// through the same chain of FMAs (one rounding each) as four vector FMAs would.  The
// instruction can take A from one of its 16 blocks (CBSZ = 4, ABID = block), so one
// register holds the coefficients of 16 such quads of slots, loaded once by 64 lanes.
// Every lane of the wavefront takes part (the matrix cores ignore EXEC): callers keep
// the wavefront together and give lanes without a point any finite coordinates.
//
// Prepared layout of one l, with nq = quads of its 2l+1 slots (U_0..U_l, V_1..V_l,
// padded with zeros): order 0 of U, V [nq][4]; then per pair of orders n = 1+2j, 2+2j
// the U, V coefficients [2][nq][4] and the W, X coefficients [2][nq][4] (zero past
// nmax).  The l's follow each other.
//
// What bounds it: VALU issue.  As vector FMAs the sums were 2420 of the 4460 VALU
// instructions per wavefront at (10, 10), issued in 83% of the cycles; a quad is one
// instruction in their place, and its 8 matrix-core cycles pass beside other wavefronts'
// recurrences and angular sums.  N = 10^6, (10, 10), potential and acceleration: 135 ->
// 93 us a call; potential only 68 -> 46 us; N = 2 10^6, (20, 14): 873 -> 472 us; N = 10^4,
// (10, 6): 25 -> 16 us.  Coefficient loads through 64-bit vector addresses kept one
// address pair per l in registers (181 VGPRs, two wavefronts per SIMD: 109 us), and
// recurrence constants through scalar loads left a wait in every pair (100 us).
//
// With T = Dual<float> (the jerk) every value carries its time derivative: a quad has a
// second accumulator, to which (coefficient) x (recurrence value)' and (coefficient)' x
// (recurrence value) go in turn, as in the Dual FMA; the derivatives of the coefficients
// are a second array of the same layout behind the first.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <int BLOCK>
__device__ __forceinline__ f32x4_t mfma_quad(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, BLOCK, 0);
}
template <int BLOCK>
__device__ __forceinline__ Dual<f32x4_t> mfma_quad(Dual<float> a, Dual<float> b, Dual<f32x4_t> c) {
  return {mfma_quad<BLOCK>(a.v, b.v, c.v), mfma_quad<BLOCK>(a.v, b.d, c.d)};
}
// the second part of a derivative's sum, apart from the first so that instructions on other
// quads stand between them
template <int BLOCK>
__device__ __forceinline__ void mfma_rest(float, float, f32x4_t&) {}
template <int BLOCK>
__device__ __forceinline__ void mfma_rest(Dual<float> a, Dual<float> b, Dual<f32x4_t>& c) {
  c.d = mfma_quad<BLOCK>(a.d, b.v, c.d);
}
template <typename T>
struct QuadOf {
  using type = f32x4_t;
  static __device__ __forceinline__ type zero() { return f32x4_t{0.f, 0.f, 0.f, 0.f}; }
  static __device__ __forceinline__ float get(const type& q, int i) { return q[i]; }
};
template <>
struct QuadOf<Dual<float>> {
  using type = Dual<f32x4_t>;
  static __device__ __forceinline__ type zero() { return {QuadOf<float>::zero(), QuadOf<float>::zero()}; }
  static __device__ __forceinline__ Dual<float> get(const type& q, int i) { return {q.v[i], q.d[i]}; }
};
__host__ __device__ constexpr int mm_quads(int l) { return slot_pad(l, 4) / 4; }
// pairs of orders from order 1 on
__host__ __device__ constexpr int mm_pairs(int nmax) { return (nmax + 1) / 2; }
// floats of the l's before l, and of the whole array (l = lmax + 1)
__host__ __device__ constexpr int mm_offset(int l, int nmax) { return zoff(l, 4) * (1 + 4 * mm_pairs(nmax)); }

template <typename T, bool ACC, int BASIS>
struct RadialMM {
  static_assert(ACC || sizeof(T) == 4, "a Dual potential alone is not instantiated");
  using Quad = typename QuadOf<T>::type;
  static constexpr bool kDual = sizeof(T) == 8;
  // The coefficients through buffer descriptors, one for each array.  A lane's position is
  // the load's vector offset, with a constant added in the instruction: both are compared
  // with the array's size, so the lanes past the values of a short run read the following
  // ones, and what lies past the array's end (the last loads of the last l, not used) is
  // zero and not read.  (A scalar offset would not be compared.)
  __amdgpu_buffer_rsrc_t cf, cd;  // cd: Dual, the derivatives
  int nmax;
  int at;                 // byte offset of this lane's value at the start of the current l
  // this lane's coefficients: order 0; the next two pairs of orders (U, V and W, X)
  T a0, x0, y0, x1, y1;

  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t array(const float* p, int values) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, 4 * values, 0x00020000);
  }
  // cfp: the prepared coefficients of one system, the same pointer in every lane
  __device__ __forceinline__ RadialMM(const float* cfp, int nmax_, int lmax_)
      : cf(array(cfp, mm_offset(lmax_ + 1, nmax_))),
        cd(array(kDual ? cfp + mm_offset(lmax_ + 1, nmax_) : cfp, mm_offset(lmax_ + 1, nmax_))), nmax(nmax_), at(0),
        a0(T(0.f)), x0(T(0.f)), y0(T(0.f)), x1(T(0.f)), y1(T(0.f)) {}

  // this lane's value `off` values on from the start of the current l
  __device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, int off) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at + 4 * off, 0, 0));
  }
  __device__ __forceinline__ T load(int off) const {
    if constexpr (kDual)
      return T(load1(cf, off), load1(cd, off));
    else
      return load1(cf, off);
  }
  // one register holds a pair's U, V and W, X quads if they are at most 16
  template <int l>
  static constexpr bool one_reg() { return ACC && 4 * mm_quads(l) <= 16; }

  // pair J of the orders of l (past the last pair: other values, not used)
  template <int l, int J>
  __device__ __forceinline__ void load_pair(T& x, T& y) const {
    constexpr int off = 4 * mm_quads(l) * (1 + 4 * J);
    x = load(off);
    if constexpr (ACC && !one_reg<l>()) y = load(off + 8 * mm_quads(l));
  }
  // the first loads of l, issued before the previous l's angular synthesis
  template <int l>
  __device__ __forceinline__ void start() {
    if constexpr (l == 0) at = 4 * int(threadIdx.x & 63);
    // opaque, so that no load's address is kept over the loop on points
    asm volatile("" : "+v"(at));
    a0 = load(0);
    load_pair<l, 0>(x0, y0);
    load_pair<l, 1>(x1, y1);
  }

  template <int l>
  __device__ __forceinline__ void sums(T xi, T (&U)[l + 1], T (&V)[l + 1], T (&W)[l + 1], T (&X)[l + 1]) {
    constexpr int NQ = mm_quads(l);
    const Quad zero = QuadOf<T>::zero();
    Quad uv[NQ], wx[NQ];
    static_for<NQ>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      uv[q] = mfma_quad<q>(a0, T(1.f), zero);
      mfma_rest<q>(a0, T(1.f), uv[q]);
    });
    T c2 = T(0.f), c1 = T(1.f);  // Chat_{n-2}, Chat_{n-1} for n = 1
    T e2 = T(0.f), e1 = T(1.f);  // Ehat_{n-2}, Ehat_{n-1}
    // order NN: c <- Chat_NN, accumulate, advance Ehat
    auto step = [&](auto nc, T x, T y, T& cA, T& cB, T& eA, T& eB) {
      constexpr int NN = decltype(nc)::value;
      constexpr int PAR = (NN - 1) % 2;
      constexpr float q = float(BASIS == kBasisCB ? kTab.qcb[l][NN] : kTab.q[l][NN]);
      constexpr float qd = float(BASIS == kBasisCB ? kTab.qdcb[l][NN] : kTab.qd[l][NN]);
      cA = recur(xi, cB, q, cA);
      static_for<NQ>([&](auto qc) {
        constexpr int b = decltype(qc)::value;
        uv[b] = mfma_quad<PAR * NQ + b>(x, cA, uv[b]);
      });
      if constexpr (ACC) {
        static_for<NQ>([&](auto qc) {
          constexpr int b = decltype(qc)::value;
          const Quad w = NN == 1 ? zero : wx[b];
          if constexpr (one_reg<l>())
            wx[b] = mfma_quad<(2 + PAR) * NQ + b>(x, eB, w);
          else
            wx[b] = mfma_quad<PAR * NQ + b>(y, eB, w);
        });
        if constexpr (kDual) {
          static_for<NQ>([&](auto qc) {
            constexpr int b = decltype(qc)::value;
            mfma_rest<PAR * NQ + b>(x, cA, uv[b]);
          });
          static_for<NQ>([&](auto qc) {
            constexpr int b = decltype(qc)::value;
            if constexpr (one_reg<l>())
              mfma_rest<(2 + PAR) * NQ + b>(x, eB, wx[b]);
            else
              mfma_rest<PAR * NQ + b>(y, eB, wx[b]);
          });
        }
        eA = recur(xi, eB, qd, eA);
      }
    };
    // The pairs are unrolled up to the cap, so the recurrence constants are literals and
    // the positions immediate offsets, with a uniform exit after each.  Every pair runs
    // both orders: past nmax (odd cutoffs) the coefficients are zero, cheaper than a
    // branch.  Two register sets take turns; a set is loaded for two pairs on as soon as
    // its pair is issued, without a condition (what lies past the last pair is not used).
    int npairs = mm_pairs(nmax);
    // opaque, so that the exit tests are compares here and not 64-bit masks kept (and
    // spilled to vector lanes) over the loop on points
    asm volatile("" : "+s"(npairs));
    auto pairs = [&](auto self, auto jc) -> void {
      constexpr int J = decltype(jc)::value;
      T& x = J % 2 ? x1 : x0;
      T& y = J % 2 ? y1 : y0;
      step(std::integral_constant<int, 1 + 2 * J>{}, x, y, c2, c1, e2, e1);
      step(std::integral_constant<int, 2 + 2 * J>{}, x, y, c1, c2, e1, e2);
      if constexpr (J + 2 < mm_pairs(NCAP)) load_pair<l, J + 2>(x, y);
      if constexpr (J + 1 < mm_pairs(NCAP)) {
        if (J + 1 < npairs) self(self, std::integral_constant<int, J + 1>{});
      }
    };
    // (no pair at nmax = 0: xi is NaN where r overflows, and times a zero coefficient it
    // would reach the monopole's potential there)
    if (npairs > 0)
      pairs(pairs, std::integral_constant<int, 0>{});
    else if constexpr (ACC)
      static_for<NQ>([&](auto qc) { wx[decltype(qc)::value] = zero; });
    at += 16 * NQ * (1 + 4 * npairs);
#pragma unroll
    for (int m = 0; m <= l; ++m) {
      U[m] = QuadOf<T>::get(uv[m / 4], m % 4);
      W[m] = QuadOf<T>::get(wx[m / 4], m % 4);
      V[m] = m > 0 ? QuadOf<T>::get(uv[(l + m) / 4], (l + m) % 4) : T(0.f);
      X[m] = m > 0 ? QuadOf<T>::get(wx[(l + m) / 4], (l + m) % 4) : T(0.f);
    }
  }
};

// Potential and acceleration at a point with spherical coordinates s; rad gives the radial
// sums (RadialF64, RadialDual, or RadialMM, whose start<0>() the caller has called)
template <typename T, int LB, bool ACC, int BASIS, typename Radial>
__device__ __forceinline__ ForceOut<T> synth_point(const Sph<T>& s, Radial& rad, int lmax) {
  using S = typename ScalarOf<T>::type;
  ForceOut<T> out{};
  {
    const T tu = s.t * s.u, u2 = s.u * s.u;
    // d/dr of the prefactor t^l u^(l+1) is l (t^l u^(l+1))/r - (2l+1) t^l u^(l+1) h, and
    // dxi/dr carries g (its constant is in the prepared coefficients):
    //   Hernquist-Ostriker h = u, g = u^2;  Clutton-Brock h = t u, g = t u^3
    const T hfac = BASIS == kBasisCB ? tu : s.u;
    const T gfac = BASIS == kBasisCB ? tu * u2 : u2;

    // cos/sin(m phi) by rotation
    T cm[LB + 1], sm[LB + 1];
    cm[0] = T(1);
    sm[0] = T(0);
#pragma unroll
    for (int m = 1; m <= LB; ++m) {
      cm[m] = sub_prod(cm[m - 1], s.cp, sm[m - 1], s.sp);
      sm[m] = add_prod(sm[m - 1], s.cp, cm[m - 1], s.sp);
    }

    // Legendre rows; row l+1 is needed for m Ybar_lm / sin(theta)
    T Y[LB + 2][LB + 2];
    Y[0][0] = T(kTab.c1[0][0]);
    auto legendre_row = [&](auto rc) {
      constexpr int r = decltype(rc)::value;
      Y[r][r] = T(kTab.c1[r][r]) * s.st * Y[r - 1][r - 1];
      Y[r][r - 1] = T(kTab.c1[r][r - 1]) * s.ct * Y[r - 1][r - 1];
      static_for<(r >= 2 ? r - 1 : 0)>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        Y[r][m] = sub_prod(T(kTab.c1[r][m]) * s.ct, Y[r - 1][m], T(kTab.c2[r][m]), Y[r - 2][m]);
      });
    };

    T accP = T(0), accR = T(0), accT = T(0), accF = T(0);
    T Rl = s.u;      // t^l u^(l+1)
    T Rprev = T(0);  // t^(l-1) u^l
    static_for<LB + 1>([&](auto lc) {
      constexpr int l = decltype(lc)::value;
      if (l > lmax) return;
      if constexpr (ACC) {
        legendre_row(std::integral_constant<int, l + 1>{});
      } else if constexpr (l >= 1) {
        legendre_row(std::integral_constant<int, l>{});
      }

      T U[l + 1], V[l + 1], W[l + 1], X[l + 1];
      rad.template sums<l>(s.xi, U, V, W, X);
      if constexpr (l < LB) {
        if (l < lmax) rad.template start<l + 1>();
      }

      // angular synthesis for this l
      T Pl = T(0), Gl = T(0), Tl = T(0), Fl = T(0);
      static_for<l + 1>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        const T ec = m >= (ACC ? l - 1 : l) ? add_prod(V[m], sm[m], U[m], cm[m]) : add_prod(U[m], cm[m], V[m], sm[m]);
        Pl = fma_(Y[l][m], ec, Pl);
        if constexpr (ACC) {
          const T gc = add_prod(W[m], cm[m], X[m], sm[m]);
          Gl = fma_(Y[l][m], gc, Gl);
          if constexpr (l >= 1) {
            T dY;
            if constexpr (m == 0) {
              dY = T(kTab.e1[l][0]) * Y[l][1];
            } else if constexpr (m + 1 <= l) {
              if constexpr (l == 2 && m == 1)  // e1 = 1
                dY = take_prod(Y[l][m + 1], T(kTab.e2[l][m]), Y[l][m - 1]);
              else
                dY = sub_prod(T(kTab.e1[l][m]), Y[l][m + 1], T(kTab.e2[l][m]), Y[l][m - 1]);
            } else {
              dY = -T(kTab.e2[l][m]) * Y[l][m - 1];
            }
            Tl = fma_(dY, ec, Tl);
            if constexpr (m >= 1) {
              const T fc = sub_prod(V[m], cm[m], U[m], sm[m]);
              const T f1 = T(kTab.f1[l][m]), f2 = T(kTab.f2[l][m]);
              // (the other product in a plain kernel's last row)
              const T mYs = l < LB || sizeof(T) != sizeof(S) ? -add_prod(f1, Y[l + 1][m + 1], f2, Y[l + 1][m - 1])
                                   : -add_prod(f2, Y[l + 1][m - 1], f1, Y[l + 1][m + 1]);
              Fl = fma_(mYs, fc, Fl);
            }
          }
        }
      });
      accP = fma_(Rl, Pl, accP);
      if constexpr (ACC) {
        const T Ql = Rprev * u2;                             // t^(l-1) u^(l+2) = (t^l u^(l+1))/r
        // d/dr (t^l u^(l+1))
        const T dRl = l == 0   ? -(Rl * hfac)
                      : l == 1 ? take_prod(Ql, T(3) * Rl, hfac)
                               : sub_prod(T(l), Ql, T(2 * l + 1) * Rl, hfac);
        T ar = l <= 1 ? add_prod(Rl * gfac, Gl, dRl, Pl) : add_prod(dRl, Pl, Rl * gfac, Gl);
        if constexpr (l == 0) {
          if (!(s.r > T(0))) ar = T(0);  // no direction at the origin
        }
        accR -= ar;
        if constexpr (l >= 1) {
          accT = take_prod(accT, Ql, Tl);
          accF = take_prod(accF, Ql, Fl);
        }
      }
      Rprev = Rl;
      Rl = Rl * tu;
    });
    out.pot = accP;
    if constexpr (ACC) {
      out.gx = take_prod(add_prod(s.st * s.cp, accR, s.ct * s.cp, accT), s.sp, accF);
      out.gy = add_prod(s.st * s.sp, accR, s.ct * s.sp, accT) + s.cp * accF;
      out.gz = sub_prod(s.ct, accR, s.st, accT);
    }
  }
  return out;
}

}  // namespace etics
