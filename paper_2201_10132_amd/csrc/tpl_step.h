// What the step kernels share (device code only): the velocity sets, storage
// access, the shifted spring term, the mixture velocity and the collisions of
// both species (Sec. V-VI).
#pragma once
#include "tpl_internal.h"

#include <type_traits>

namespace tplk {

// ---------------------------------------------------------------------------
// Velocity sets.
// D2Q9 (Sec. VI.A; the standard set, the only one matching the weights
// 4/9, 1/9, 1/36).
constexpr int C9X[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int C9Y[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
constexpr double W9[9] = {4.0 / 9,  1.0 / 9,  1.0 / 9,  1.0 / 9, 1.0 / 9,
                          1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// D4Q25 (Sec. VI.B, Table I) as (v_x, v_y, Qdot_x, Qdot_y): the rest vector,
// then for the coordinate pairs (vx,vy) (vx,Qx) (vx,Qy) (vy,Qx) (vy,Qy)
// (Qx,Qy) the sign pairs (+,+) (+,-) (-,+) (-,-).
constexpr int PV[25][4] = {
    {0, 0, 0, 0},                                                    //
    {1, 1, 0, 0},  {1, -1, 0, 0},  {-1, 1, 0, 0},  {-1, -1, 0, 0},   //
    {1, 0, 1, 0},  {1, 0, -1, 0},  {-1, 0, 1, 0},  {-1, 0, -1, 0},   //
    {1, 0, 0, 1},  {1, 0, 0, -1},  {-1, 0, 0, 1},  {-1, 0, 0, -1},   //
    {0, 1, 1, 0},  {0, 1, -1, 0},  {0, -1, 1, 0},  {0, -1, -1, 0},   //
    {0, 1, 0, 1},  {0, 1, 0, -1},  {0, -1, 0, 1},  {0, -1, 0, -1},   //
    {0, 0, 1, 1},  {0, 0, 1, -1},  {0, 0, -1, 1},  {0, 0, -1, -1}};  //

// D2Q9 direction of a D4Q25 velocity's r-part.
__host__ __device__ constexpr int dir9(int vx, int vy) {
  return (vx == 0 && vy == 0)    ? 0
         : (vx == 1 && vy == 0)  ? 1
         : (vx == 0 && vy == 1)  ? 2
         : (vx == -1 && vy == 0) ? 3
         : (vx == 0 && vy == -1) ? 4
         : (vx == 1 && vy == 1)  ? 5
         : (vx == -1 && vy == 1) ? 6
         : (vx == -1 && vy == -1) ? 7
                                  : 8;
}
__host__ __device__ constexpr int pdir(int k) { return dir9(PV[k][0], PV[k][1]); }
// The D4Q25 velocities grouped by r-direction: those of direction d are
// KDIR[KDIR0[d]] .. KDIR[KDIR0[d + 1] - 1].
constexpr int KDIR[25] = {0,  21, 22, 23, 24, 5,  6,  9,  10, 13, 14, 17, 18,
                          7,  8,  11, 12, 15, 16, 19, 20, 1,  3,  4,  2};
constexpr int KDIR0[10] = {0, 5, 9, 13, 17, 21, 22, 23, 24, 25};
// The velocity with the same r-part and reversed Q-part (Q bounce-back).
__host__ __device__ constexpr int kstar(int k) {
  int j = 0;
  for (int i = 0; i < 25; ++i)
    if (PV[i][0] == PV[k][0] && PV[i][1] == PV[k][1] &&
        PV[i][2] == -PV[k][2] && PV[i][3] == -PV[k][3])
      j = i;
  return j;
}
static_assert(kstar(5) == 6 && kstar(21) == 24 && kstar(22) == 23 &&
                  kstar(1) == 1 && pdir(9) == 1 && pdir(16) == 4,
              "D4Q25 table");
__host__ __device__ constexpr bool kdir_grouped() {
  for (int d = 0; d < 9; ++d)
    for (int i = KDIR0[d]; i < KDIR0[d + 1]; ++i)
      if (pdir(KDIR[i]) != d) return false;
  return true;
}
static_assert(kdir_grouped(), "velocities by r-direction");
// Opposite velocities: -c_d (D2Q9) and -(v_k, Qdot_k) (D4Q25).
__host__ __device__ constexpr int rev9(int d) {
  return dir9(-C9X[d], -C9Y[d]);
}
__host__ __device__ constexpr int krev(int k) {
  int j = 0;
  for (int i = 0; i < 25; ++i)
    if (PV[i][0] == -PV[k][0] && PV[i][1] == -PV[k][1] && PV[i][2] == -PV[k][2] &&
        PV[i][3] == -PV[k][3])
      j = i;
  return j;
}
static_assert(rev9(1) == 3 && rev9(5) == 7 && rev9(8) == 6 && krev(0) == 0 && krev(1) == 4 &&
                  krev(5) == 8 && krev(21) == 24 && krev(13) == 16,
              "opposite velocities");

__device__ __forceinline__ int xcd_tile(int bid, int tiles_per_xcd) {
  // Workgroups are dispatched round-robin over the 8 XCDs; give each XCD a
  // contiguous range of tiles so that stencil neighbours share its L2.
  return tiles_per_xcd > 0 ? (bid & 7) * tiles_per_xcd + (bid >> 3) : bid;
}

// ---------------------------------------------------------------------------
// Storage access.  Loads and stores at a wave-uniform plane base plus a 32-bit
// byte offset (every offset is < sizeof(T) N < 2^32).  The base goes through
// readfirstlane so that it stays in scalar registers; the compiler hoists the
// zero-extended offsets out of the Q-loop and issues the accesses with 64-bit
// per-lane addresses (SGPR base plus offset, one VALU add each).  Forcing the
// SGPR-base instruction form instead (an opaque 32-bit offset per access)
// saves 8-15 VGPRs but measured no faster: the step is bound by DRAM.
template <typename T>
__device__ __forceinline__ T *uni(T *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T *>(((uint64_t)hi << 32) | lo);
}
// Accesses go through the global address space explicitly: a generic
// (flat) pointer would force 64-bit per-lane addresses and FLAT instructions.
#define GLOBAL_AS __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T ldo(const T *base, uint32_t off) {
  const char GLOBAL_AS *b = (const char GLOBAL_AS *)(base);
  return *(const T GLOBAL_AS *)(b + off);
}
template <typename T>
__device__ __forceinline__ void sto(T *base, uint32_t off, T v) {
  char GLOBAL_AS *b = (char GLOBAL_AS *)(base);
  *(T GLOBAL_AS *)(b + off) = v;
}
// Read-only tables (reference values, instance records) are read through the
// constant address space, which the compiler turns into scalar loads whenever
// the address is wave-uniform.
#define CONSTANT_AS __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const T CONSTANT_AS *cst(const T *p) {
  return (const T CONSTANT_AS *)(p);
}

// Full value from a stored one: identity for FP64, reference + deviation for
// the FP32 form (ref = the plane's reference value at this row).
__device__ __forceinline__ double full(double v, double) { return v; }
__device__ __forceinline__ double full(float v, double ref) { return ref + (double)v; }
template <typename T>
__device__ __forceinline__ T stored(double v, double ref);
template <>
__device__ __forceinline__ double stored<double>(double v, double) { return v; }
template <>
__device__ __forceinline__ float stored<float>(double v, double ref) { return (float)(v - ref); }

// BF16 form: a polymer population is stored as the BF16 rounding (nearest
// even) of its deviation from the FP32 reference, the x-invariant base state;
// solvent and psi keep FP32 deviations.  BF16 has FP32's exponent range, so
// the deviations need no scaling.
// Rounds two FP32 values in one instruction, a to the lower half.
__device__ __forceinline__ uint32_t to_bf16_pair(float a, float b) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), h2));
}
// One value.  (The empty asm hides where it comes from: the compiler would
// fuse an FP64-to-FP32 rounding before it into one rounding to BF16, another
// value; it does not do so with pairs, where the asm costs 20 % of the step.)
__device__ __forceinline__ uint16_t to_bf16(float v) {
  asm("" : "+v"(v));
  return __builtin_bit_cast(uint16_t, (__bf16)v);
}
__device__ __forceinline__ double from_bf16(uint16_t b) {
  return (double)__uint_as_float(((uint32_t)b) << 16);
}

// ---------------------------------------------------------------------------
// Non-local spring term: psi(r + Q/2) - psi(r - Q/2) of one Q-node's plane P
// (stored T, FP32 reference rpq(row)) at node (x, y), each side by bilinear
// interpolation between its four surrounding nodes, periodic.  The Q-node's
// offsets are wave-uniform; the wrap loops run at most NQ/4 + 1 times (a
// narrow lattice such as the one-column base-state run wraps more than once).
__device__ __forceinline__ int wrap_to(int v, int n) {
  while (v < 0) v += n;
  while (v >= n) v -= n;
  return v;
}
template <typename T, typename RefRow>
__device__ __forceinline__ double spring_shift_diff(const T *P, int x, int y, int nx, int ny,
                                                   double qx, double qy, RefRow rpq) {
#pragma clang fp contract(off)
  const double ax = 0.5 * qx, ay = 0.5 * qy;
  const double flx = floor(ax), fly = floor(ay);
  const double fx = ax - flx, fy = ay - fly;
  const int ix = (int)flx, iy = (int)fly;
  auto at = [&](int xx, int yy) {
    return full(ldo(P, (uint32_t)sizeof(T) * (uint32_t)(yy * nx + xx)), rpq(yy));
  };
  // + side: floor(Q/2) and the next node; - side: floor(-Q/2) = -floor(Q/2) - 1
  // (Q/2 is never an integer: Q-nodes sit at half-integers), weights swapped
  int xp0, xp1, yp0, yp1, xm0, xm1, ym0, ym1;
  if ((ix < 0 ? -ix : ix) + 2 <= nx && (iy < 0 ? -iy : iy) + 2 <= ny) {
    // offsets shorter than the lattice (wave-uniform test): every index lies
    // in [-n, 2n), one conditional add or subtract wraps it
    auto wr = [](int v, int n) {
      v = v < 0 ? v + n : v;
      return v >= n ? v - n : v;
    };
    xp0 = wr(x + ix, nx); xp1 = wr(x + ix + 1, nx);
    yp0 = wr(y + iy, ny); yp1 = wr(y + iy + 1, ny);
    xm0 = wr(x - ix - 1, nx); xm1 = wr(x - ix, nx);
    ym0 = wr(y - iy - 1, ny); ym1 = wr(y - iy, ny);
  } else {
    xp0 = wrap_to(x + ix, nx); xp1 = wrap_to(x + ix + 1, nx);
    yp0 = wrap_to(y + iy, ny); yp1 = wrap_to(y + iy + 1, ny);
    xm0 = wrap_to(x - ix - 1, nx); xm1 = wrap_to(x - ix, nx);
    ym0 = wrap_to(y - iy - 1, ny); ym1 = wrap_to(y - iy, ny);
  }
  const double w00 = (1.0 - fx) * (1.0 - fy), w10 = fx * (1.0 - fy);
  const double w01 = (1.0 - fx) * fy, w11 = fx * fy;
  const double vp = fma(w11, at(xp1, yp1), fma(w01, at(xp0, yp1),
                        fma(w00, at(xp0, yp0), w10 * at(xp1, yp0))));
  const double vm = fma(w00, at(xm1, ym1), fma(w10, at(xm0, ym1),
                        fma(w11, at(xm0, ym0), w01 * at(xm1, ym0))));
  return vp - vm;
}

// The arithmetic below is written with explicit fused multiply-adds and no
// contraction by the compiler, so that every kernel that uses it rounds alike
// (which of two products the compiler would fuse depends on the code around).
// The last bit matters: the FP32 and BF16 forms round small deviations, and a
// last-bit change upstream flips a few per cent of those roundings.

// Mixture velocity: the velocity at which the momentum exchange of the two
// species cancels (Sec. IV/V), from their g-momenta, the body force and the
// Q-sum S of the spring term, weighted by 1 / (2 tJ + 1) per species; den is
// the densities' sum with the same weights.
__device__ __forceinline__ void mixture_velocity(const StepParams &p, double den, double JSx,
                                                 double JSy, double JPx, double JPy,
                                                 double Sx, double Sy, double Fbx, double Fby,
                                                 double &Ux, double &Uy) {
#pragma clang fp contract(off)
  Ux = fma(JPx + Sx / (2.0 * p.tJP), p.aP, fma(0.5, Fbx, JSx) * p.aS) / den;
  Uy = fma(JPy + Sy / (2.0 * p.tJP), p.aP, fma(0.5, Fby, JSy) * p.aS) / den;
}

// Taylor form of the spring term: Q . grad psi by central differences.
__device__ __forceinline__ double spring_taylor(double qx, double qy, double pE, double pW,
                                                double pN, double pS) {
#pragma clang fp contract(off)
  return fma(qx, 0.5 * (pE - pW), qy * (0.5 * (pN - pS)));
}

// Solvent collision of one node: relaxes the pulled gS (moments rhoS, JS)
// towards its equilibria about the mixture velocity U under the body force
// Fb, hands each post-collision population to put(d, value) and returns their
// momentum.
template <bool QE2, typename Put>
__device__ __forceinline__ void solvent_collide(const StepParams &p, const double (&gS)[9],
                                                double rhoS, double JSx, double JSy, double Ux,
                                                double Uy, double Fbx, double Fby, Put put,
                                                double &jx, double &jy) {
#pragma clang fp contract(off)
  // model 1: f* about the species' own (inverted) momentum; model 2: f*
  // with the equilibrium's momentum and the species' own (inverted) stress
  const double vx = Ux + p.tJS * Fbx / rhoS, vy = Uy + p.tJS * Fby / rhoS;
  const double v2 = fma(vy, vy, vx * vx);
  double usx = 0.0, usy = 0.0, Dxx = 0.0, Dxy = 0.0, Dyy = 0.0;
  if constexpr (!QE2) {
    usx = fma(p.tJS, Fbx, fma(2.0 * p.tJS, JSx, rhoS * Ux)) * p.aS / rhoS;
    usy = fma(p.tJS, Fby, fma(2.0 * p.tJS, JSy, rhoS * Uy)) * p.aS / rhoS;
  } else {
    // P(f) - rho c_s^2 I with P(f) = (2 tau2 P(g) + rho (c_s^2 I + v v)) / (2 tau2 + 1)
    double Pxx = 0.0, Pxy = 0.0, Pyy = 0.0;
#pragma unroll
    for (int d = 0; d < 9; ++d) {
      if (C9X[d]) Pxx += gS[d];
      if (C9Y[d]) Pyy += gS[d];
      if (C9X[d] && C9Y[d]) Pxy += C9X[d] * C9Y[d] * gS[d];
    }
    const double t2 = 1.0 - p.pS;  // 2 tau2 / (2 tau2 + 1)
    Dxx = fma(t2, Pxx, p.pS * rhoS * fma(vx, vx, 1.0 / 3.0)) - rhoS / 3.0;
    Dyy = fma(t2, Pyy, p.pS * rhoS * fma(vy, vy, 1.0 / 3.0)) - rhoS / 3.0;
    Dxy = fma(t2, Pxy, p.pS * rhoS * vx * vy);
  }
  const double us2 = fma(usy, usy, usx * usx);
  jx = 0.0;
  jy = 0.0;
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    const double cv = C9X[d] * vx + C9Y[d] * vy;
    const double fe = W9[d] * rhoS * (fma(cv, 4.5 * cv, fma(3.0, cv, 1.0)) - 1.5 * v2);
    double fs;
    if constexpr (!QE2) {
      const double cu = C9X[d] * usx + C9Y[d] * usy;
      fs = W9[d] * rhoS * (fma(cu, 4.5 * cu, fma(3.0, cu, 1.0)) - 1.5 * us2);
    } else {  // second-order Hermite form with the stress D + rho c_s^2 I
      const double cxx = C9X[d] * C9X[d] - 1.0 / 3.0, cyy = C9Y[d] * C9Y[d] - 1.0 / 3.0;
      double h;
      if (C9X[d] && !C9Y[d]) h = fma(cxx, Dxx, cyy * Dyy);
      else if (C9Y[d] && !C9X[d]) h = fma(cyy, Dyy, cxx * Dxx);
      else h = cxx * Dxx + cyy * Dyy;
      if (C9X[d] && C9Y[d]) h += 2.0 * Dxy * C9X[d] * C9Y[d];
      fs = W9[d] * fma(4.5, h, fma(3.0 * rhoS, cv, rhoS));
    }
    const double o = fma(p.c1S, gS[d], p.c2S * fma(p.rS, fe, (1.0 - p.rS) * fs));
    if (C9X[d]) jx += C9X[d] * o;
    if (C9Y[d]) jy += C9Y[d] * o;
    put(d, o);
  }
}

// Moments of one (r, Q)-node's pulled populations G(k), k = 0..24: density,
// r- and Q-momentum, and for model 2 the second moments sum xi_a xi_b g
// (a <= b).
template <bool QE2>
struct PolyMoments {
  double psi = 0.0, Jrx = 0.0, Jry = 0.0, JQx = 0.0, JQy = 0.0;
  double P2[4][4] = {};
};
template <bool QE2, typename Pop>
__device__ __forceinline__ PolyMoments<QE2> polymer_moments(Pop G) {
#pragma clang fp contract(off)
  PolyMoments<QE2> m;
#pragma unroll
  for (int k = 0; k < 25; ++k) {
    const double gk = G(k);
    m.psi += gk;
    if (PV[k][0]) m.Jrx += PV[k][0] * gk;
    if (PV[k][1]) m.Jry += PV[k][1] * gk;
    if (PV[k][2]) m.JQx += PV[k][2] * gk;
    if (PV[k][3]) m.JQy += PV[k][3] * gk;
    if constexpr (QE2) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b2 = a; b2 < 4; ++b2)
          if (PV[k][a] && PV[k][b2]) m.P2[a][b2] += PV[k][a] * PV[k][b2] * gk;
    }
  }
  return m;
}

// The relaxation target c2 [(1 - r) f* + r f_eq] of one (r, Q)-node, built
// from its moments, the imposed fluxes (mixture velocity U, its gradient K,
// spring term (sx, sy), Q-node position and force) and the moment inversion;
// term(k) is its value for velocity k (post-collision = c1 g + term).
template <bool QE2>
struct PolyTarget {
  double psi, c2w0, c2w1, w3, one_r, hw, trD3;
  double A[4];
  double P2[4][4];

  __device__ __forceinline__ PolyTarget(const StepParams &p, const PolyMoments<QE2> &m, double Ux,
                                        double Uy, double Kxx, double Kxy, double Kyx, double Kyy,
                                        double sx, double sy, double qx, double qy, double fx,
                                        double fy) {
#pragma clang fp contract(off)
    psi = m.psi;
    c2w0 = p.c2P * (1.0 / 3.0);
    c2w1 = p.c2P * (1.0 / 36.0);
    one_r = 1.0 - p.rP;
    const double Erx = fma(psi, Ux, sx), Ery = fma(psi, Uy, sy);
    const double EQx = psi * fma(-p.DQ, fx, fma(Kxx, qx, Kxy * qy));
    const double EQy = psi * fma(-p.DQ, fy, fma(Kyx, qx, Kyy * qy));
    if constexpr (!QE2) {
      const double Frx = fma(2.0 * p.tJP, m.Jrx, Erx) * p.aP;
      const double Fry = fma(2.0 * p.tJP, m.Jry, Ery) * p.aP;
      const double FQx = fma(2.0 * p.tJP, m.JQx, EQx) * p.aP;
      const double FQy = fma(2.0 * p.tJP, m.JQy, EQy) * p.aP;
      // (1 - r) f* + r f_eq is the linear equilibrium of the blended fluxes
      A[0] = fma(p.rP, Erx, one_r * Frx);
      A[1] = fma(p.rP, Ery, one_r * Fry);
      A[2] = fma(p.rP, EQx, one_r * FQx);
      A[3] = fma(p.rP, EQy, one_r * FQy);
    } else {
      // f* and f_eq share the imposed fluxes; f* adds the Hermite term of
      // D = P(f) - psi c_s^2 I, P(f) = (2 tau2 P(g) + psi c_s^2 I) / (2 tau2 + 1)
      A[0] = Erx;
      A[1] = Ery;
      A[2] = EQx;
      A[3] = EQy;
      const double t2 = 1.0 - p.pP;
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        P2[a][a] = fma(t2, m.P2[a][a], p.pP * psi / 3.0) - psi / 3.0;
#pragma unroll
        for (int b2 = a + 1; b2 < 4; ++b2) P2[a][b2] = m.P2[a][b2] * t2;
      }
    }
    w3 = 3.0 * c2w1;
    // model 2: the Hermite term's factor c2 (1 - r) 4.5 w_k, and -tr(D)/3
    hw = 4.5 * one_r * c2w1;
    trD3 = QE2 ? (P2[0][0] + P2[1][1] + P2[2][2] + P2[3][3]) / 3.0 : 0.0;
  }

  __device__ __forceinline__ double term(int k) const {
#pragma clang fp contract(off)
    // w (psi + 3 xi . A): every moving velocity has two unit entries a < b
    if (k == 0) {
      const double t = c2w0 * psi;
      return QE2 ? fma(c2w0, psi, -(4.5 * one_r * c2w0 * trD3)) : t;
    }
    const int a0 = PV[k][0] ? 0 : PV[k][1] ? 1 : 2;
    const int b0 = PV[k][3] ? 3 : PV[k][2] ? 2 : 1;
    double t = fma(PV[k][b0] * w3, A[b0], fma(c2w1, psi, PV[k][a0] * (w3 * A[a0])));
    if constexpr (QE2) {
      // sum_ab D_ab (xi_a xi_b - delta_ab / 3)
      const double hk =
          fma(2.0 * PV[k][a0] * PV[k][b0], P2[a0][b0], P2[a0][a0] - trD3) + P2[b0][b0];
      t = fma(hw, hk, t);
    }
    return t;
  }
};

// The instance of a batch that an item (64-node tile) belongs to: the last one
// with item0 <= item.
__device__ __forceinline__ int batch_instance(const InstDev CONSTANT_AS *ci, int ninst,
                                              int item) {
  int lo = 0, hi = ninst - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ci[mid].item0 <= item) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// An instance's step parameters.  Field-by-field reads through the constant
// address space keep every value in SGPRs (a whole-struct copy would go
// through private memory).
__device__ __forceinline__ StepParams batch_params(const InstDev CONSTANT_AS &d, bool qe2) {
  StepParams pp;
#define TPL_LD(f) pp.f = d.p.f;
  TPL_LD(nx) TPL_LD(ny) TPL_LD(nqd) TPL_LD(qs) TPL_LD(ntiles) TPL_LD(tiles_per_xcd)
  TPL_LD(y0) TPL_LD(N) TPL_LD(aS) TPL_LD(aP) TPL_LD(tJS) TPL_LD(tJP) TPL_LD(c1S)
  TPL_LD(c2S) TPL_LD(rS) TPL_LD(c1P) TPL_LD(c2P) TPL_LD(rP) TPL_LD(kappa) TPL_LD(DQ)
  TPL_LD(F0) TPL_LD(kf) TPL_LD(src)
#undef TPL_LD
  pp.wg = 0;
  pp.gate = nullptr;
  pp.qe = qe2 ? 2 : 1;
  pp.shift = 0;
  pp.pS = qe2 ? d.p.pS : 0.0;
  pp.pP = qe2 ? d.p.pP : 0.0;
  return pp;
}

}  // namespace tplk
