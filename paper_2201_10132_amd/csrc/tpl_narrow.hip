// The fused step for lattices of few nodes (small lattices, the one-column
// base state): a workgroup of eight waves holds NPW nodes instead of 64, its
// lanes are (node, Q-node) pairs, so that a lattice of N nodes fills N / NPW
// workgroups and every workgroup works on 8 * 64 / NPW Q-nodes at a time.
//
// It computes, bit for bit, what step_tile computes with eight Q-slices: wave
// w holds slice w (Q-nodes w, w + 8, w + 16, ...), and the slice's sums over
// its Q-nodes are formed in the same order, lane group after lane group.
//
// What bounds it: the misses that one CU keeps in flight.  A node's Q-disk is
// nqd * 400 bytes in and out, a CU gets about 45 GB/s of lines that another
// CU wrote in the step before, and with 64 nodes per wave a 64^2 lattice is 64
// workgroups on 256 CUs (a 256-row column 4), so the split goes for more CUs
// first.  16 nodes are one 128-byte line of FP64 values per plane; 4 nodes
// waste three quarters of each line and pay only where CUs are idle otherwise
// (1 x 256, NQ 16: 97 us with 64 nodes per wave, 35 with 16, 29 with 8, 24
// with 4; 64^2, NQ 16: 161, 81, 114, 165).  Before that bound the pass was
// serial: table, then populations, then about 200 dependent FP64 operations;
// the next pass's loads and the table row after it are therefore issued
// before a pass computes (39 to 33 us), and the slice sums go through LDS
// once per pass instead of lane group by lane group.
#include "tpl_step.h"

namespace tplk {

constexpr int kNarrowWaves = 8;  // the Q-slices of step_tile's widest split
constexpr int kNarrowLds = kNarrowWaves * 29 * 64;

// Orders a wave's LDS writes before the reads of its other lanes (LDS
// operations of one wave complete in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One group of NPW consecutive nodes.  red: LDS of kNarrowLds doubles.
template <typename T, bool B16, bool QE2, bool SHIFT, int NPW>
__device__ __forceinline__ void step_narrow(const StepParams &p, const StateT<T> &a,
                                            const StateT<T> &b, const float *__restrict__ rpull,
                                            const float *__restrict__ rstore,
                                            const float *__restrict__ rpsi,
                                            const float *__restrict__ rspull,
                                            const float *__restrict__ rsstore,
                                            const QNode *__restrict__ qtab, const int group,
                                            double *red) {
  constexpr bool F32 = std::is_same<T, float>::value;
  constexpr uint32_t SZ = sizeof(T);
  constexpr int GROUPS = 64 / NPW;              // lane groups, one Q-node each
  constexpr int QPP = kNarrowWaves * GROUPS;    // Q-nodes of the workgroup per pass
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & (NPW - 1), lg = lane / NPW;
  const long long N = p.N;
  const long long rr = (long long)group * NPW + n;
  const bool active = rr < N;
  const int r = (int)(active ? rr : N - 1);
  const int nx = p.nx, ny = p.ny, nqd = p.nqd;
  const int y = r / nx, x = r - y * nx;
  const int xm = (x == 0) ? nx - 1 : x - 1, xp = (x == nx - 1) ? 0 : x + 1;
  const int ym = (y == 0) ? ny - 1 : y - 1, yp = (y == ny - 1) ? 0 : y + 1;
  const uint32_t rE = (uint32_t)(y * nx + xp), rW = (uint32_t)(y * nx + xm);
  const uint32_t rN = (uint32_t)(yp * nx + x), rS = (uint32_t)(ym * nx + x);
  const uint32_t fR = 8u * (uint32_t)r;
  uint32_t src[9];  // node index of the pull source r - c_d
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    const int sx = C9X[d] == 1 ? xm : (C9X[d] == -1 ? xp : x);
    const int sy = C9Y[d] == 1 ? ym : (C9Y[d] == -1 ? yp : y);
    src[d] = (uint32_t)(sy * nx + sx);
  }
  auto fplane = [&](const double *arr, int i) { return uni(arr + (size_t)i * N); };
  auto wfplane = [&](double *arr, int i) { return uni(arr + (size_t)i * N); };
  auto rq = [&](const float *tab, int q, int k) -> double {
    return F32 ? (double)cst(tab)[((size_t)y * nqd + q) * 25 + k] : 0.0;
  };
  auto rpq = [&](int row, int q) -> double {
    return F32 ? (double)cst(rpsi)[(size_t)row * nqd + q] : 0.0;
  };
  auto rsd = [&](const float *tab, int d) -> double {
    return F32 ? (double)cst(tab)[(size_t)y * 9 + d] : 0.0;
  };

  // A (node, Q-node) pair as pulled: stored populations and the lagged psi of
  // the four neighbours.  Loaded one pass ahead of its use.
  using RT = std::conditional_t<B16, uint16_t, T>;
  constexpr int NR = B16 ? 26 : 25;
  struct Pulled {
    RT g[NR];
    T psi[4];
    double qx, qy, fx, fy;
  };
  // the whole population array is below 2^32 bytes and a plane below 2^24, so
  // an address is one 24-bit multiply-add on a wave-uniform base
  const uint32_t pb = (uint32_t)sizeof(RT) * (uint32_t)N, sb = SZ * (uint32_t)N;
  // the table's source planes of a Q-node come another pass earlier, or every
  // pass would wait for them before it can issue its loads
  int pl[25];
  auto clamped = [&](int q) { return q < nqd ? q : nqd - 1; };
  auto planes = [&](int q) {
    const QNode CONSTANT_AS &qn = cst(qtab)[q];
#pragma unroll
    for (int k = B16 ? 1 : 0; k < 25; ++k) pl[k] = qn.plane[k];
  };
  auto load = [&](int q, Pulled &v) {  // pl holds q's planes
    const QNode CONSTANT_AS &qn = cst(qtab)[q];
    v.qx = qn.qx;
    v.qy = qn.qy;
    v.fx = qn.fx;
    v.fy = qn.fy;
    const RT *XP = reinterpret_cast<const RT *>(a.XP);
    auto at = [&](int plane, uint32_t node) {
      return ldo(XP, __umul24((uint32_t)plane, pb) + (uint32_t)sizeof(RT) * node);
    };
    if constexpr (B16) {  // the rest population's two halves: planes 0 and 25
      v.g[0] = at(q, (uint32_t)r);
      v.g[25] = at(25 * nqd + q, (uint32_t)r);
    }
#pragma unroll
    for (int k = B16 ? 1 : 0; k < 25; ++k) v.g[k] = at(pl[k], src[pdir(k)]);
    if constexpr (!SHIFT) {
      const uint32_t P = __umul24((uint32_t)q, sb);
      v.psi[0] = ldo(a.PSI, P + SZ * rE);
      v.psi[1] = ldo(a.PSI, P + SZ * rW);
      v.psi[2] = ldo(a.PSI, P + SZ * rN);
      v.psi[3] = ldo(a.PSI, P + SZ * rS);
    }
  };
  const int q0 = kNarrowWaves * lg + wave;  // this lane's Q-node of pass 0
  Pulled cur, nxt;
  planes(clamped(q0));
  load(clamped(q0), cur);
  if (QPP < nqd) planes(clamped(q0 + QPP));

  // ---- solvent, streamed Q-marginals, lagged non-local terms, mixture
  // velocity: as in step_tile, by every lane
  double gS[9], rhoS = 0.0, JSx = 0.0, JSy = 0.0;
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    gS[d] = full(ldo(uni(a.XS + (size_t)d * N), SZ * src[d]), rsd(rspull, d));
    rhoS += gS[d];
    if (C9X[d]) JSx += C9X[d] * gS[d];
    if (C9Y[d]) JSy += C9Y[d] * gS[d];
  }
  double rhoP = 0.0, JPx = 0.0, JPy = 0.0;
#pragma unroll
  for (int d = 0; d < 9; ++d) {
    const double m = ldo(fplane(a.FLD, F_M0 + d), 8u * src[d]);
    rhoP += m;
    if (C9X[d]) JPx += C9X[d] * m;
    if (C9Y[d]) JPy += C9Y[d] * m;
  }
  auto dX = [&](int f) {
    return 0.5 * (ldo(fplane(a.FLD, f), 8u * rE) - ldo(fplane(a.FLD, f), 8u * rW));
  };
  auto dY = [&](int f) {
    return 0.5 * (ldo(fplane(a.FLD, f), 8u * rN) - ldo(fplane(a.FLD, f), 8u * rS));
  };
  const double Kxx = dX(F_UX), Kxy = dY(F_UX), Kyx = dX(F_UY), Kyy = dY(F_UY);
  const double Sx = SHIFT ? ldo(fplane(a.FLD, F_MXX), fR) : p.kappa * (dX(F_MXX) + dY(F_MXY));
  const double Sy = SHIFT ? ldo(fplane(a.FLD, F_MXY), fR) : p.kappa * (dX(F_MXY) + dY(F_MYY));
  double Fbx = p.F0 * sin(p.kf * (double)(y + p.y0)), Fby = 0.0;
  if (p.src != nullptr) {
    Fbx += p.src[r];
    Fby = p.src[N + r];
  }
  double Ux, Uy;
  mixture_velocity(p, fma(rhoS, p.aS, rhoP * p.aP), JSx, JSy, JPx, JPy, Sx, Sy, Fbx, Fby, Ux,
                   Uy);

  // the last wave collides the solvent and writes the fields known by now
  if (wave == kNarrowWaves - 1) {
    const bool writer = active && lg == 0;
    double jx, jy;
    solvent_collide<QE2>(p, gS, rhoS, JSx, JSy, Ux, Uy, Fbx, Fby,
                         [&](int d, double o) {
                           if (writer)
                             sto(uni(b.XS + (size_t)d * N), SZ * (uint32_t)r,
                                 stored<T>(o, rsd(rsstore, d)));
                         },
                         jx, jy);
    if (writer) {
      sto(wfplane(b.FLD, F_JSX), fR, jx);
      sto(wfplane(b.FLD, F_JSY), fR, jy);
      sto(wfplane(b.FLD, F_RHOS), fR, rhoS);
      sto(wfplane(b.FLD, F_RHOP), fR, rhoP);
      sto(wfplane(b.FLD, F_UX), fR, Ux);
      sto(wfplane(b.FLD, F_UY), fR, Uy);
    }
  }

  // ---- polymer: one Q-node per lane group and pass
  // The wave's slice sums (9 marginals, then M): each lane holds NSUM of the
  // 12 NPW (component, node) pairs, pair i of lane l being l + 64 i.
  constexpr int NSUM = (12 * NPW + 63) / 64;
  double sum[NSUM];
#pragma unroll
  for (int i = 0; i < NSUM; ++i) sum[i] = 0.0;
  double *mine = red + wave * 29 * 64;  // [25 velocities, psi Q, Fhat][lane groups][NPW]
  for (int base = 0; base < nqd; base += QPP) {
    const int q = base + q0;
    const bool valid = q < nqd;
    const int qc = clamped(q);  // idle lanes of the last pass repeat the last Q-node
    if (base + QPP < nqd) {
      load(clamped(q + QPP), nxt);
      if (base + 2 * QPP < nqd) planes(clamped(q + 2 * QPP));
    }
    const double qx = cur.qx, qy = cur.qy, fx = cur.fx, fy = cur.fy;
    double g[25];
#pragma unroll
    for (int k = 0; k < 25; ++k) {
      if constexpr (B16)
        g[k] = rq(rpull, qc, k) +
               (k == 0 ? (double)__uint_as_float(((uint32_t)cur.g[0] << 16) | cur.g[NR - 1])
                       : from_bf16(cur.g[k]));
      else
        g[k] = full(cur.g[k], rq(rpull, qc, k));
    }
    const PolyMoments<QE2> m = polymer_moments<QE2>([&](int k) { return g[k]; });
    const double psi = m.psi;
    double qg;
    if constexpr (SHIFT) {
      qg = spring_shift_diff(a.PSI + (size_t)qc * N, x, y, nx, ny, qx, qy,
                             [&](int row) { return rpq(row, qc); });
    } else {
      const double pE = full(cur.psi[0], rpq(y, qc)), pW = full(cur.psi[1], rpq(y, qc));
      const double pN = full(cur.psi[2], rpq(yp, qc)), pS = full(cur.psi[3], rpq(ym, qc));
      qg = spring_taylor(qx, qy, pE, pW, pN, pS);
    }
    const double sx = p.kappa * fx * qg, sy = p.kappa * fy * qg;
    const PolyTarget<QE2> target(p, m, Ux, Uy, Kxx, Kxy, Kyx, Kyy, sx, sy, qx, qy, fx, fy);
#pragma unroll
    for (int i = 0; i < 25; ++i) {
      g[KDIR[i]] = fma(p.c1P, g[KDIR[i]], target.term(KDIR[i]));
      mine[i * 64 + lane] = g[KDIR[i]];
    }
    mine[25 * 64 + lane] = psi * qx;
    mine[26 * 64 + lane] = psi * qy;
    mine[27 * 64 + lane] = fx;
    mine[28 * 64 + lane] = fy;
    wave_lds_sync();
    if (active && valid) {
      const uint32_t w = __umul24((uint32_t)q, pb) + (uint32_t)sizeof(RT) * (uint32_t)r;
      RT *XP = reinterpret_cast<RT *>(b.XP);
      auto plane = [&](int k) { return uni(XP + (size_t)k * nqd * N); };
      if constexpr (!B16) {
#pragma unroll
        for (int k = 0; k < 25; ++k)
          sto(plane(k), w, stored<T>(g[k], rq(rstore, qc, k)));
      } else {
        // deviations rounded to BF16; the rest population in FP32 with the
        // rounding residual of the others, over planes 0 and 25
        float res = 0.0f, dv0 = 0.0f;
#pragma unroll
        for (int k = 0; k < 25; ++k) {
          const float dv = (float)(g[k] - rq(rstore, qc, k));
          if (k == 0) {
            dv0 = dv;
          } else {
            const uint16_t h = to_bf16(dv);
            res += dv - (float)from_bf16(h);
            sto(plane(k), w, h);
          }
        }
        const uint32_t u0 = __float_as_uint(dv0 + res);
        sto(plane(0), w, (uint16_t)(u0 >> 16));
        sto(plane(25), w, (uint16_t)(u0 & 0xffffu));
      }
      sto(b.PSI, __umul24((uint32_t)q, sb) + SZ * (uint32_t)r, stored<T>(psi, rpq(y, qc)));
    }
    // add the pass's terms to the slice sums, lane group (Q-node) after lane
    // group: the order in which one wave walking the slice adds them
#pragma unroll
    for (int i = 0; i < NSUM; ++i) {
      const int j = lane + 64 * i, c = j / NPW;
      if (j >= 12 * NPW) break;
      // component c's velocities: terms and first LDS row (KDIR0[c])
      const int terms = c == 0 ? 5 : c < 5 ? 4 : c < 9 ? 1 : 0;
      const int row = c == 0 ? 0 : c < 5 ? 1 + 4 * c : 16 + c;
      const int most = i * GROUPS == 0 ? 5 : i * GROUPS < 5 ? 4 : 1;  // of this i
#pragma unroll
      for (int gq = 0; gq < GROUPS; ++gq) {
        const bool in = base + kNarrowWaves * gq + wave < nqd;  // wave-uniform
        const int at = gq * NPW + (j & (NPW - 1));
#pragma unroll
        for (int t = 0; t < most; ++t) {
          const bool has = t < terms;
          const double v = mine[(has ? row + t : 0) * 64 + at];
          sum[i] += in && has ? v : 0.0;
        }
        if ((i + 1) * GROUPS > 9) {  // M = sum psi Q Fhat^T: xx, xy, yy
          const double v = mine[(c == 11 ? 26 : 25) * 64 + at];
          sum[i] = fma(in && c >= 9 ? v : 0.0, mine[(c == 9 ? 27 : 28) * 64 + at], sum[i]);
        }
      }
    }
    wave_lds_sync();  // before the next pass overwrites the terms
    cur = nxt;
  }

  // ---- combine the slices' sums in slice order
  __syncthreads();  // red changes its layout
#pragma unroll
  for (int i = 0; i < NSUM; ++i)
    if (lane + 64 * i < 12 * NPW) red[wave * 12 * NPW + lane + 64 * i] = sum[i];
  __syncthreads();
  for (int i = threadIdx.x; i < 12 * NPW; i += 64 * kNarrowWaves) {
    double v = red[i];
    for (int s = 1; s < kNarrowWaves; ++s) v += red[s * 12 * NPW + i];
    const int c = i / NPW;
    const long long node = (long long)group * NPW + (i & (NPW - 1));
    const int f = c < 9 ? F_M0 + c : F_MXX + c - 9;
    if (node < N) b.FLD[(size_t)f * N + node] = v;
  }
}

template <typename T, bool B16, bool QE2, bool SHIFT, int NPW>
__global__ void __launch_bounds__(64 * kNarrowWaves)
    k_step_narrow(StepParams p, StateT<T> a, StateT<T> b, const float *__restrict__ rpull,
                  const float *__restrict__ rstore, const float *__restrict__ rpsi,
                  const float *__restrict__ rspull, const float *__restrict__ rsstore,
                  const QNode *__restrict__ qtab, int ngroups, int per_xcd) {
  __shared__ double red[kNarrowLds];
  if (p.gate && *p.gate) return;  // a learned correction's drift gate closed
  const int group = xcd_tile(blockIdx.x, per_xcd);
  if (group >= ngroups) return;  // whole workgroup leaves together
  step_narrow<T, B16, QE2, SHIFT, NPW>(p, a, b, rpull, rstore, rpsi, rspull, rsstore, qtab, group,
                                       red);
}

// The kernel's 24-bit plane strides and 32-bit offsets (8-byte elements and
// the BF16 form's 26 planes cover every form).
static bool narrow_fits(long long N, int nqd) {
  return 8 * N < (1 << 24) && 26 * (long long)nqd < (1 << 24) && 26 * 8 * nqd * N < (1LL << 32);
}
static bool narrow_small(long long N, int nqd) { return N <= kNarrowSmall && nqd > 32; }

template <typename T, bool B16, int NPW>
hipError_t launch_narrow(const StepParams &p, StateT<T> a, StateT<T> b, const StepRef &r,
                         const QNode *qtab, hipStream_t s) {
  const int ngroups = (int)((p.N + NPW - 1) / NPW);
  const int per_xcd = ngroups >= 64 ? (ngroups + 7) / 8 : 0;
  const dim3 grid(per_xcd > 0 ? 8 * per_xcd : ngroups), blk(64 * kNarrowWaves);
#define TPL_NARROW(QE2, SHIFT)                                                                  \
  hipLaunchKernelGGL((k_step_narrow<T, B16, QE2, SHIFT, NPW>), grid, blk, 0, s, p, a, b, r.pull, \
                     r.store, r.psi, r.spull, r.sstore, qtab, ngroups, per_xcd)
  if constexpr (B16) {
    if (p.qe == 2) TPL_NARROW(true, false); else TPL_NARROW(false, false);
  } else {
    if (p.shift) {
      if (p.qe == 2) TPL_NARROW(true, true); else TPL_NARROW(false, true);
    } else {
      if (p.qe == 2) TPL_NARROW(true, false); else TPL_NARROW(false, false);
    }
  }
#undef TPL_NARROW
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step_narrow(const StepParams &p, StateT<T> a, StateT<T> b, StepRef r,
                              const QNode *qtab, hipStream_t s, bool b16) {
  if (p.qs != kNarrowWaves || p.wg || (p.qe != 1 && p.qe != 2)) return hipErrorInvalidValue;
  if (!narrow_fits(p.N, p.nqd)) return hipErrorInvalidValue;
  if constexpr (std::is_same<T, float>::value) {
    if (b16)
      return p.shift ? hipErrorInvalidValue : launch_narrow<T, true, 16>(p, a, b, r, qtab, s);
  } else {
    if (b16) return hipErrorInvalidValue;
    if (narrow_small(p.N, p.nqd)) return launch_narrow<T, false, 4>(p, a, b, r, qtab, s);
  }
  return launch_narrow<T, false, 16>(p, a, b, r, qtab, s);
}
template hipError_t launch_step_narrow<double>(const StepParams &, StateT<double>, StateT<double>,
                                               StepRef, const QNode *, hipStream_t, bool);
template hipError_t launch_step_narrow<float>(const StepParams &, StateT<float>, StateT<float>,
                                              StepRef, const QNode *, hipStream_t, bool);

// The same for every instance of a batch: 64 / kNarrowNodes workgroups per
// item (64-node tile); parity selects the half read as in k_step_batch.
template <typename T, bool QE2, bool SHIFT, int NPW>
__global__ void __launch_bounds__(64 * kNarrowWaves)
    k_step_batch_narrow(const InstDev *__restrict__ inst, int ninst, int ngroups, int per_xcd,
                        int parity) {
  __shared__ double red[kNarrowLds];
  constexpr int SUB = 64 / NPW;
  const int unit = xcd_tile(blockIdx.x, per_xcd);
  if (unit >= ngroups) return;
  const int item = unit / SUB;
  const InstDev CONSTANT_AS &d = cst(inst)[batch_instance(cst(inst), ninst, item)];
  const StepParams pp = batch_params(d, QE2);
  const int group = (item - d.item0) * SUB + unit % SUB;
  if ((long long)group * NPW >= pp.N) return;  // past the last node of a ragged tile
  const int rd = parity ^ d.cur0;
  const StateT<T> a{static_cast<T *>(d.XS[rd]), static_cast<T *>(d.XP[rd]),
                    static_cast<T *>(d.PSI[rd]), d.FLD[rd]};
  const StateT<T> b{static_cast<T *>(d.XS[rd ^ 1]), static_cast<T *>(d.XP[rd ^ 1]),
                    static_cast<T *>(d.PSI[rd ^ 1]), d.FLD[rd ^ 1]};
  step_narrow<T, false, QE2, SHIFT, NPW>(pp, a, b, d.rpull, d.rstore, d.rpsi, d.rspull, d.rsstore,
                                         d.qtab, group, red);
}

template <typename T, int NPW>
hipError_t launch_batch_narrow(const InstDev *inst, int ninst, int nitems, int parity,
                               hipStream_t s, bool shift, bool qe2) {
  const int ngroups = nitems * (64 / NPW);
  const int per_xcd = ngroups >= 64 ? (ngroups + 7) / 8 : 0;
  const dim3 grid(per_xcd > 0 ? 8 * per_xcd : ngroups), blk(64 * kNarrowWaves);
#define TPL_NARROW(QE2, SHIFT)                                                              \
  hipLaunchKernelGGL((k_step_batch_narrow<T, QE2, SHIFT, NPW>), grid, blk, 0, s, inst, ninst, \
                     ngroups, per_xcd, parity)
  if (shift) TPL_NARROW(false, true);
  else if (qe2) TPL_NARROW(true, false);
  else TPL_NARROW(false, false);
#undef TPL_NARROW
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step_batch_narrow(const InstDev *inst, int ninst, int nitems, int nqd,
                                    int parity, hipStream_t s, bool shift, bool qe2) {
  if (nitems < 1 || (shift && qe2) || !narrow_fits(64LL * nitems, nqd))
    return hipErrorInvalidValue;
  if constexpr (std::is_same<T, double>::value)
    if (narrow_small(64LL * nitems, nqd))
      return launch_batch_narrow<T, 4>(inst, ninst, nitems, parity, s, shift, qe2);
  return launch_batch_narrow<T, 16>(inst, ninst, nitems, parity, s, shift, qe2);
}
template hipError_t launch_step_batch_narrow<double>(const InstDev *, int, int, int, int,
                                                     hipStream_t, bool, bool);
template hipError_t launch_step_batch_narrow<float>(const InstDev *, int, int, int, int,
                                                    hipStream_t, bool, bool);

}  // namespace tplk
