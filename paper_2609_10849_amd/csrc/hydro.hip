// Hydrodynamic-subflow kernels for gfx950 (section "Hydrodynamic subflow: entropy-stable DGSEM").
//
// The flux-differencing volume term uses the skew form sum_{r != i} S_ir F(U_i, U_r) (S = Q - Q^T),
// which equals eq. euler-volume-residual combined with the boundary corrections of
// eq. euler-nodal-index; each unordered pair of a line is evaluated once.  The stage kernel gives a
// thread a whole grid line of an element, so that the pairs' operands, both halves of each flux
// and the coefficients stay in registers.  Reductions are in fixed order, so results are
// deterministic run to run.
#include <cfloat>

#include "common.h"
#include "xcd.h"
#include "ec_log.h"
#include "jumps.h"
#include "rsqrt.h"

// Every fused operation of this file is written out.  Left to the compiler, which product of a sum it fuses
// differs between instantiations of one kernel; a run's results are the same bit for bit for every tile and
// every form of a kernel that it can take, alone and in a batch.
#pragma clang fp contract(off)

namespace {

constexpr double EPSM = 2.220446049250313e-16;  // 2^-52

template <int P, int BS = 256>
struct Cfg {
  static constexpr int NP = P + 1, NN = NP * NP, EB = BS / NN, NT = EB * NN;
};

// node values of the EC flux: density, half velocities (normal to the line's direction first) and the
// ratio rho / p (twice the inverse temperature beta)
struct Prim {
  double r, hn, ht, hz, b;
};

// Logarithmic means (eq. euler-chandrashekar-flux) of near values without logarithms: with
// f = (aR - aL) / (aR + aL) and z = f^2 the mean is (aL + aR)/2 G(z), G(z) = f / atanh f, and its reciprocal
// 2/(aL + aR) H(z), H(z) = atanh f / f = 1 + z/3 + z^2/5 + ...; G's coefficients are those of 1/H.  Both
// series are summed to z^7: for |f| <= LM_NEAR = 0.1 (values within 22 % of each other) the first omitted
// term is below 1.2e-18 (G) and 6e-18 (H) relative.  The coefficients come from the tables, as scalars (as
// literals each costs two register moves).
constexpr double LM_NEAR = 0.1;
__device__ __forceinline__ double lm_series(const double* __restrict__ c, double z) {
  double s = c[LM_N - 1];
#pragma unroll
  for (int k = LM_N - 2; k >= 0; --k) s = fma(s, z, c[k]);
  return fma(s, z, 1.0);
}

// Logarithmic mean of any two values as a fraction num/den, from the values a and their logarithms l.
// Well separated (f^2 >= 1e-4): (aR-aL)/(lR-lL).  Near-equal: with x = (lR-lL)/2 = atanh f, the mean is
// (aL+aR) tanh(x) / (2x) = (aL+aR) / (2 x coth x), and 2 x coth x = 2 + y/6 - y^2/360 + y^3/15120 - ...
// in y = (lR-lL)^2 (the Laurent series of coth); there y < 4.1e-4, so the first omitted term is below
// 1e-19 relative.
struct Frac {
  double n, d;
};
__device__ __forceinline__ Frac lmean_frac(double aL, double aR, double lL, double lR) {
  const double d = aR - aL, s = aR + aL, dl = lR - lL;
  const double y = dl * dl;
  const double pu = fma(y, fma(-y, fma(-y, 1.0 / 15120.0, 1.0 / 360.0), 1.0 / 6.0), 2.0);
  const bool near = d * d < 1e-4 * (s * s);
  return Frac{near ? s : d, near ? pu : dl};
}

// Chandrashekar flux (eq. euler-chandrashekar-flux) in the line's frame (mass, normal, tangential and
// z momentum, energy) from the logarithmic mean rl of rho, the reciprocal one ibl of b = rho / p and
// ph = (rhoL + rhoR) / (bL + bR).  With half velocities h = u / 2 the averages are plain sums, and
// |avg u|^2 - avg |u|^2 / 2 = u_L . u_R / 2 = 2 h_L . h_R; 1 / (2 (g-1) beta_log) = cg / b_log, cg = 1/(g-1).
__device__ __forceinline__ void ec_form(const Prim& L, const Prim& R, double rl, double ibl, double ph, double cg,
                                        double F[5]) {
  const double un = L.hn + R.hn, ut = L.ht + R.ht, uz = L.hz + R.hz;
  const double f0 = rl * un;
  const double dot = dot3(L.hn, L.ht, L.hz, R.hn, R.ht, R.hz);
  F[0] = f0;
  F[1] = fma(f0, un, ph);
  F[2] = f0 * ut;
  F[3] = f0 * uz;
  F[4] = fma(f0, fma(ibl, cg, 2.0 * dot), ph * un);
}
// near values: one reciprocal for the three quotients
__device__ __forceinline__ void ecflux_near(const Prim& L, const Prim& R, double cg, const HydroTab* __restrict__ T,
                                            double F[5]) {
  const double sr = L.r + R.r, sb = L.b + R.b;
  const double is = rcp_refined(sr * sb), isb = sr * is;
  const double fr = (R.r - L.r) * (sb * is), fb = (R.b - L.b) * isb;
  const double G = lm_series(T->lmG, fr * fr), H = lm_series(T->lmH, fb * fb);
  ec_form(L, R, 0.5 * sr * G, (isb + isb) * H, sr * isb, cg, F);
}
// any values, with their logarithms (lr of rho, lb of b)
__device__ __forceinline__ void ecflux_log(const Prim& L, double lrL, double lbL, const Prim& R, double lrR, double lbR,
                                           double cg, double F[5]) {
  const Frac fr = lmean_frac(L.r, R.r, lrL, lrR);
  const Frac fb = lmean_frac(L.b, R.b, lbL, lbR);
  const double sb = L.b + R.b;
  const double t1 = fr.d * fb.n;
  const double Q = rcp_refined(t1 * sb);  // nonzero: each factor is a positive sum or a nonzero difference
  const double sq = sb * Q;
  ec_form(L, R, fr.n * fb.n * sq, fb.d * fr.d * sq, (L.r + R.r) * (t1 * Q), cg, F);
}

// pressure of a conserved state whose reciprocal density is ir
__device__ __forceinline__ double pressure_of(const double U[5], double ir, double g) {
  return (g - 1.0) * fma(-0.5 * ir, dot3(U[1], U[2], U[3], U[1], U[2], U[3]), U[4]);
}

// One side of an LLF interface flux (eq. euler-lf-flux) in the line's frame from density, half
// velocities and pressure: conserved values, physical flux and wave speed |u_n| + c.
struct FaceSide {
  double U[5], F[5], s;
};
__device__ __forceinline__ FaceSide face_side(double r, double hn, double ht, double hz, double p, double g,
                                              double cg) {
  FaceSide a;
  const double un = hn + hn, x = g * p * rcp_refined(r);  // squared sound speed, positive
  const double y = rsqrt_refined(x), c0 = x * y;
  const double c = fma(0.5 * y, fma(-c0, c0, x), c0);  // sqrt(x)
  a.U[0] = r; a.U[1] = r * un; a.U[2] = r * (ht + ht); a.U[3] = r * (hz + hz);
  a.U[4] = fma(cg, p, 2.0 * r * dot3(hn, ht, hz, hn, ht, hz));
  a.F[0] = a.U[1];
  a.F[1] = fma(a.U[1], un, p);
  a.F[2] = a.U[2] * un;
  a.F[3] = a.U[3] * un;
  a.F[4] = (a.U[4] + p) * un;
  a.s = fabs(un) + c;
  return a;
}

// Interface flux of a line's end node q (pressure pq) with its neighbour's conserved values n, the minus side at -1
// (side 0) and the plus side at +1: LLF, or (iface 1) the EC flux
__device__ __forceinline__ void face_flux(const Prim& q, double pq, const double n[5], int D, int side, int iface, double g,
                                          double cg, double F[5]) {
  const double ir = rcp_refined(n[0]), hi = 0.5 * ir, pn = pressure_of(n, ir, g);
  const double hn = (D ? n[2] : n[1]) * hi, ht = (D ? n[1] : n[2]) * hi, hz = n[3] * hi;
  if (iface == 1) {
    const Prim o{n[0], hn, ht, hz, n[0] * rcp_refined(pn)};
    ecflux_log(q, log_ec(q.r), log_ec(q.b), o, log_ec(o.r), log_ec(o.b), cg, F);
    return;
  }
  const FaceSide a = face_side(q.r, q.hn, q.ht, q.hz, pq, g, cg), b = face_side(n[0], hn, ht, hz, pn, g, cg);
  const double hl = (side ? -0.5 : 0.5) * fmax(a.s, b.s);
#pragma unroll
  for (int c = 0; c < 5; ++c) F[c] = fma(0.5, a.F[c] + b.F[c], hl * (b.U[c] - a.U[c]));
}

// Face f = 2 D + side of element (ex, ey) (D 0: the x-normal faces, D 1: the y-normal faces; side 0
// is the face at -1) and the face node `line` on it: the neighbour element en across the face, the
// element's own face node qo and the neighbour's node qn at the same point (periodic mesh).
template <int P>
__device__ __forceinline__ void face_match(const MeshP& mp, int ex, int ey, int D, int side, int line, int& en,
                                           int& qo, int& qn) {
  constexpr int NP = P + 1;
  const int pos = side ? P : 0;
  qo = D == 0 ? line * NP + pos : pos * NP + line;
  qn = D == 0 ? line * NP + (P - pos) : (P - pos) * NP + line;
  en = D == 0 ? ey * mp.nx + wrap32(ex + (side ? 1 : -1), mp.nx) : wrap32(ey + (side ? 1 : -1), mp.ny) * mp.nx + ex;
}

// does a line (its nodes at r and b, step apart) hold values too far apart for the series of the logarithmic mean?
template <int P>
__device__ __forceinline__ bool line_far(const double* r, const double* b, int step) {
  double r0 = r[0], r1 = r0, b0 = b[0], b1 = b0;
#pragma unroll
  for (int i = 1; i <= P; ++i) {
    const double x = r[i * step], y = b[i * step];
    r0 = x < r0 ? x : r0; r1 = x > r1 ? x : r1;
    b0 = y < b0 ? y : b0; b1 = y > b1 ? y : b1;
  }
  return !(r1 - r0 <= LM_NEAR * (r1 + r0)) || !(b1 - b0 <= LM_NEAR * (b1 + b0));
}

// Element statistics of five fields in LDS (component c at v + c row, element el at el ES, node (i, j) at j RS + i):
// weighted sum (without |J_K|), minimum and maximum of each component to stats, and the raw-average
// admissibility (NaN-safe) to flag (may be null).  ssum: 5 nel free values.  All threads of the block must call this.
template <int P, int BS, int RS, int ES>
__device__ __forceinline__ void stage_stats(const double* v, int row, double* ssum, int e0, int nel,
                                            double* __restrict__ stats, int* __restrict__ flag,
                                            const HydroTab* __restrict__ T, double g) {
  constexpr int NP = P + 1;
  const int tid = threadIdx.x;
  for (int t = tid; t < nel * 5; t += BS) {
    const int es = t / 5, c = t - es * 5;
    const double* f = v + c * row + es * ES;
    double s = 0.0, mn = f[0], mx = f[0];
#pragma unroll 1
    for (int j = 0; j < NP; ++j) {
      double sr = 0.0;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double x = f[j * RS + i];
        sr = fma(T->w[i], x, sr);
        mn = fmin(mn, x); mx = fmax(mx, x);
      }
      s = fma(T->w[j], sr, s);
    }
    double* o = stats + ((long)(e0 + es) * 5 + c) * 3;
    o[0] = s; o[1] = mn; o[2] = mx;
    ssum[t] = s;
  }
  if (!flag) return;
  __syncthreads();
  if (tid < nel) {
    double a[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) a[c] = 0.25 * ssum[tid * 5 + c];
    const double pb = (g - 1.0) * (a[4] - dot3(a[1], a[2], a[3], a[1], a[2], a[3]) / (2.0 * a[0]));
    if (!(a[0] > 0.0) || !(pb > 0.0)) atomicOr(flag, 1);
  }
}

// Tile of the stage kernel: the x lines of EB elements on the block's first half, their y lines on
// the second (so a wave has one direction), EB = (BS / 2) / (p+1).  An element's node arrays in LDS keep
// rows of odd stride RS, so that both the row and the column reads spread over the banks.
template <int P, int BS>
struct SC {
  static constexpr int NP = P + 1, NN = NP * NP, EB = BS / 2 / NP, RS = NP | 1, ES = NP * RS;
};

// MODE 0: out = L_E(Us).  MODE 1: out = ca*Un + cb*(Us + tau*L_E(Us)) plus element statistics.
//
// Phases: (1) per node, the values of the EC flux into LDS, and which lines need logarithms; (2) per
// line, its two interface fluxes and its p(p+1)/2 pair fluxes, the coefficients as scalars and the
// residual of the line in registers; (3) the x lines' residuals into LDS over the node values, the y
// lines' added; (4) per node, the SSP combine; (5) per element and component, the statistics.
// A thread per node instead (each pair's second half through LDS, coefficients and partners by run-time
// index, two logarithms per node) issued 4.3e8 VALU instructions a launch at 1024^2, N = 4 and was bound
// by that: 1.02 ms.  This form issues 2.2e8, takes 0.82 ms and moves 4.2 GB (5 TB/s, a large copy's
// rate), 1.4 times its arrays, the excess all reads (U_s is read twice, and its face nodes by the neighbours); at
// 512^2, N = 3 0.160 -> 0.131 ms, at 256^2, N = 2 31.5 -> 21.8 us.  Four waves per SIMD: at three it takes 0.87 ms.
// N = 4 fits 117 registers, with 36 bytes of scratch a lane and 6 spilled scalars; N = 5 and 6 need 133 and 145 (three
// waves), the same scratch and 22 and 34 spilled scalars.
template <int P, int MODE, int BS>
__device__ __forceinline__ void hydro_stage_body(const double* __restrict__ Us, const double* __restrict__ Un,
                                                    double* __restrict__ out, double* __restrict__ stats,
                                                    int* __restrict__ flag, const HydroTab* __restrict__ T, MeshP mp,
                                                    double ca, double cb, double tau, int iface, long blk) {
  using C = SC<P, BS>;
  constexpr int NP = C::NP, NN = C::NN, EB = C::EB, RS = C::RS, ES = C::ES;
  __shared__ double sp[8][EB * ES];  // rho, h_x, h_y, h_z, b, p, log rho, log b; rows 0..4 later the residual
  __shared__ int sflag;
  const int tid = threadIdx.x;
  const int e0 = (int)(blk * EB);
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;
  const long KN = mp.K * NN;
  const double cg = 2.0 * mp.gk;
  auto slot = [](int n) {  // LDS slot of the block's n-th node
    const int el = n / NN, q = n - el * NN, j = q / NP;
    return el * ES + j * RS + (q - j * NP);
  };
  // every global load of the line phase is issued before the first wait (the reject word's too: read
  // once per block, because other blocks may set it)
  constexpr int NR = (EB * NN + BS - 1) / BS;  // nodes per thread
  double U[NR][5];
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int n = tid + m * BS;
    const unsigned no = ((unsigned)e0 * NN + n) * 8u;  // the node's byte offset in a component array
    if (n < nel * NN) {
#pragma unroll
      for (int c = 0; c < 5; ++c) U[m][c] = bld(node_rsrc(Us + c * KN, KN), no);
    }
  }
  // the thread's line: direction D (0: x, 1: y, the same for a wave), element el, line ln
  const int D = __builtin_amdgcn_readfirstlane(tid >= BS / 2 ? 1 : 0);
  const int lt = tid - D * (BS / 2), el = lt / NP, ln = lt - el * NP;
  const bool act = lt < nel * NP;
  const int base = el * ES + (D ? ln : ln * RS), step = D ? RS : 1;  // LDS slots of the line's nodes
  // the neighbours' face nodes (index 0: the face at -1, 1: at +1)
  double nb[2][5];
  if (act) {
    int ex, ey;
    elem_xy32(mp, e0 + el, ex, ey);
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      int en, qo, qn;
      face_match<P>(mp, ex, ey, D, side, ln, en, qo, qn);
      const unsigned on = ((unsigned)en * NN + qn) * 8u;
#pragma unroll
      for (int c = 0; c < 5; ++c) nb[side][c] = bld(node_rsrc(Us + c * KN, KN), on);
    }
  }
  if (MODE == 1 && tid == 0) sflag = __atomic_load_n(flag, __ATOMIC_RELAXED);
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int n = tid + m * BS;
    if (n < nel * NN) {
      const double* u = U[m];
      const double ir = rcp_refined(u[0]), hi = 0.5 * ir;  // rho > 0 on admissible states
      const double p = pressure_of(u, ir, mp.gamma);
      const int k = slot(n);
      sp[0][k] = u[0]; sp[1][k] = u[1] * hi; sp[2][k] = u[2] * hi; sp[3][k] = u[3] * hi;
      sp[4][k] = u[0] * rcp_refined(p); sp[5][k] = p;  // p > 0 on admissible states
    }
  }
  __syncthreads();
  if (MODE == 1 && sflag) return;  // skip stages after a rejected one
  double acc[NP][5];
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int c = 0; c < 5; ++c) acc[i][c] = 0.0;
  const int rn = 1 + D, rt = 2 - D;  // LDS rows of the normal and the tangential velocity / momentum
  auto node = [&](int i) {
    const int k = base + i * step;
    return Prim{sp[0][k], sp[rn][k], sp[rt][k], sp[3][k], sp[4][k]};
  };
  // Each line answers for itself whether its pairs take the series, so that a pair's arithmetic depends on its own
  // line's values only, not on which elements share the block
  const bool lfar = act && line_far<P>(sp[0] + base, sp[4] + base, step);
  if (__syncthreads_or(lfar)) {  // then the block's node logarithms, which its far lines read
    for (int n = tid; n < nel * NN; n += BS) {
      const int k = slot(n);
      sp[6][k] = log_ec(sp[0][k]);
      sp[7][k] = log_ec(sp[4][k]);
    }
    __syncthreads();
  }
  if (act) {
    // interface fluxes
    const double rw = rcp_refined(T->w[0]);
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const int i = side ? P : 0;
      double F[5];
      face_flux(node(i), sp[5][base + i * step], nb[side], D, side, iface, mp.gamma, cg, F);
#pragma unroll
      for (int c = 0; c < 5; ++c) acc[i][c] = fma(side ? rw : -rw, F[c], acc[i][c]);
    }
    // S_ir by its exact symmetry S_{p-i,p-r} = -S_ir (the tables hold it bit for bit), which halves the
    // scalars that the pairs keep
    auto S = [&](int i, int r) {
      return i * NP + r <= (P - i) * NP + (P - r) ? T->Shat[i][r] : -T->Shat[P - i][P - r];
    };
    // the partner is read again for every pair: LDS reads are cheap here, and with a whole line's values
    // in registers the kernel fits one wave per SIMD less
    auto pairs = [&](auto flux) {
#pragma unroll
      for (int i = 0; i + 1 < NP; ++i) {
#pragma unroll
        for (int r = i + 1; r < NP; ++r) {
          double F[5];
          flux(i, r, F);
          const double si = S(i, r), sr = S(r, i);
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            acc[i][c] = fma(si, F[c], acc[i][c]);
            acc[r][c] = fma(sr, F[c], acc[r][c]);
          }
          SCHED_FENCE();
        }
      }
    };
    if (__builtin_expect(lfar, 0)) {
      pairs([&](int i, int r, double* F) {
        const int ki = base + i * step, kr = base + r * step;
        ecflux_log(node(i), sp[6][ki], sp[7][ki], node(r), sp[6][kr], sp[7][kr], cg, F);
      });
    } else {
      pairs([&](int i, int r, double* F) { ecflux_near(node(i), node(r), cg, T, F); });
    }
    const double sc = -2.0 * (D ? mp.rhy : mp.rhx);
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
      for (int c = 0; c < 5; ++c) acc[i][c] *= sc;
  }
  __syncthreads();  // every line has read its values; the residual overwrites rows 0..4
  if (act) {
    if (D == 0) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int k = base + i * step;
#pragma unroll
        for (int c = 0; c < 5; ++c) sp[c][k] = acc[i][c];
      }
    }
  }
  // the node values of the combine are loaded before the barrier, so that their latency overlaps it; it
  // is carried as (ca U^n + cb U_s) + cb tau L; the first stage (ca = 0) has no U^n term
  double Y[NR][5];
  if (MODE == 1) {
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = tid + m * BS;
      const unsigned no = ((unsigned)e0 * NN + n) * 8u;
      if (n < nel * NN) {
#pragma unroll
        for (int c = 0; c < 5; ++c) Y[m][c] = cb * bld(node_rsrc(Us + c * KN, KN), no);
        if (ca != 0.0) {
#pragma unroll
          for (int c = 0; c < 5; ++c) Y[m][c] = fma(ca, bld(node_rsrc(Un + c * KN, KN), no), Y[m][c]);
        }
      }
    }
  }
  __syncthreads();
  if (act && D == 1) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int k = base + i * step;
      sp[0][k] += acc[i][0]; sp[2][k] += acc[i][1]; sp[1][k] += acc[i][2];
      sp[3][k] += acc[i][3]; sp[4][k] += acc[i][4];
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int n = tid + m * BS;
    if (n < nel * NN) {
      const unsigned no = ((unsigned)e0 * NN + n) * 8u;
      const int k = slot(n);
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        if (MODE == 0) {
          bst(node_rsrc(out + c * KN, KN), no, sp[c][k]);
        } else {
          const double v = fma(cb * tau, sp[c][k], Y[m][c]);
          bst(node_rsrc(out + c * KN, KN), no, v);
          sp[c][k] = v;
        }
      }
    }
  }
  if (MODE == 0) return;
  __syncthreads();
  stage_stats<P, BS, RS, ES>(sp[0], EB * ES, sp[5], e0, nel, stats, flag, T, mp.gamma);
}

template <int P, int MODE, int BS>
__global__ __launch_bounds__(BS, 4) void k_hydro_stage(const double* __restrict__ Us, const double* __restrict__ Un,
                                                    double* __restrict__ out, double* __restrict__ stats,
                                                    int* __restrict__ flag, const HydroTab* __restrict__ T, MeshP mp,
                                                    double ca, double cb, double tau, int iface) {
  hydro_stage_body<P, MODE, BS>(Us, Un, out, stats, flag, T, mp, ca, cb, tau, iface, xcd_block());
}

struct hydro_stage_args {
  const double* Us;
  const double* Un;
  double* out;
  double* stats;
  int* flag;
  const HydroTab* T;
  MeshP mp;
  double ca;
  double cb;
  double tau;
  int iface;
};

template <int P, int MODE, int BS>
__global__ __launch_bounds__(BS, 4) void k_hydro_stage_rt(const hydro_stage_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const hydro_stage_args& a = A[r];
  hydro_stage_body<P, MODE, BS>(gl(a.Us), gl(a.Un), gl(a.out), gl(a.stats), gl(a.flag), gl(a.T), a.mp, a.ca, a.cb, a.tau, a.iface, (long)blockIdx.x - boff[r]);
}

// The stage on small meshes (see small_mesh): a thread per node, EB elements per block, the same arithmetic.  In the
// form above a line's thread works through its p(p+1)/2 pairs one after another, and that is the time of a launch with
// fewer blocks than the chip has places.  Here the pairs of all lines, then the face nodes, are tasks spread over the
// element's threads, their fluxes go through LDS, and each node adds its own in the line's order.  At 16^2 elements it
// takes 6.9 (N = 3), 7.3 (4), 7.9 (5), 8.8 us (6) where the form above takes 7.7, 9.8, 12.0, 13.2; at 48^2 8.6, 11.4,
// 17.0, 19.8 against 8.1, 10.1, 12.4, 14.3.
template <int P, int MODE, int BS>
__device__ __forceinline__ void hydro_stage_node_body(const double* __restrict__ Us, const double* __restrict__ Un,
                                                      double* __restrict__ out, double* __restrict__ stats,
                                                      int* __restrict__ flag, const HydroTab* __restrict__ T, MeshP mp,
                                                      double ca, double cb, double tau, int iface, long blk) {
  constexpr int NP = P + 1, NN = NP * NP, EB = BS / (2 * NN), TPE = BS / EB, NPR = NP * P / 2, RS = NP, ES = NN;
  __shared__ double sp[8][EB * ES];             // as above
  __shared__ double sF[EB][2][NP][NPR][5];      // pair fluxes [direction][line][pair][component in the line's frame]
  __shared__ double sG[EB][2][2][NP][5];        // interface fluxes [direction][side][line][component]
  __shared__ unsigned char sfar[EB][2][NP], sa[NPR], sb[NPR];  // far lines; a pair's nodes
  static_assert(NN + 4 * NP <= TPE, "the face nodes have threads of their own");
  __shared__ int sflag;
  auto pair = [](int i, int r) { return i * NP - i * (i + 1) / 2 + r - i - 1; };  // index of the pair i < r
  const int tid = threadIdx.x, el = tid / TPE, q = tid - el * TPE;
  const int e0 = (int)(blk * EB), e = e0 + el;
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;
  const bool act = el < nel, own = act && q < NN;  // own: the thread has node q
  const int k = el * NN + q;                          // its slot
  const long KN = mp.K * NN;
  const unsigned no = ((unsigned)e * NN + q) * 8u;  // the node's byte offset in a component array
  const double cg = 2.0 * mp.gk;
  // the thread's face node (direction, side, line) and its node's rows of S; with the node's own values and the
  // neighbour's all global loads are issued before the first wait
  const int fq0 = q - NN, fD = fq0 / (2 * NP), fside = fq0 / NP & 1, fln = fq0 % NP;
  const bool face = act && fq0 >= 0 && fq0 < 4 * NP;
  int fq = 0;
  double Y[5], n[5], S[2][NP];
  if (face) {
    int ex, ey, en, qn;
    elem_xy32(mp, e, ex, ey);
    face_match<P>(mp, ex, ey, fD, fside, fln, en, fq, qn);
#pragma unroll
    for (int c = 0; c < 5; ++c) n[c] = bld(node_rsrc(Us + c * KN, KN), ((unsigned)en * NN + qn) * 8u);
  }
  if (own) {
    double U[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) U[c] = bld(node_rsrc(Us + c * KN, KN), no);
#pragma unroll
    for (int r = 0; r < NP; ++r) { S[0][r] = T->Shat[q % NP][r]; S[1][r] = T->Shat[q / NP][r]; }
    if (MODE == 1) {
#pragma unroll
      for (int c = 0; c < 5; ++c) Y[c] = cb * U[c];
      if (ca != 0.0) {
#pragma unroll
        for (int c = 0; c < 5; ++c) Y[c] = fma(ca, bld(node_rsrc(Un + c * KN, KN), no), Y[c]);
      }
    }
    const double ir = rcp_refined(U[0]), hi = 0.5 * ir, p = pressure_of(U, ir, mp.gamma);
    sp[0][k] = U[0]; sp[1][k] = U[1] * hi; sp[2][k] = U[2] * hi; sp[3][k] = U[3] * hi;
    sp[4][k] = U[0] * rcp_refined(p); sp[5][k] = p;
  }
  if (tid < NN) {
    const int i = tid / NP, r = tid - i * NP;
    if (i < r) { sa[pair(i, r)] = i; sb[pair(i, r)] = r; }
  }
  if (MODE == 1 && tid == 0) sflag = __atomic_load_n(flag, __ATOMIC_RELAXED);
  __syncthreads();
  if (MODE == 1 && sflag) return;  // skip stages after a rejected one
  // the far lines (task = element, direction, line)
  bool lfar = false;
  for (int t = tid; t < nel * 2 * NP; t += BS) {
    const int es = t / (2 * NP), D = t / NP & 1, ln = t % NP, base = es * ES + (D ? ln : ln * RS);
    const bool f = line_far<P>(sp[0] + base, sp[4] + base, D ? RS : 1);
    sfar[es][D][ln] = f;
    lfar = lfar || f;
  }
  if (__syncthreads_or(lfar)) {
    if (own) {
      sp[6][k] = log_ec(sp[0][k]);
      sp[7][k] = log_ec(sp[4][k]);
    }
    __syncthreads();
  }
  auto node = [&](int k, int D) { return Prim{sp[0][k], sp[1 + D][k], sp[2 - D][k], sp[3][k], sp[4][k]}; };
  if (act) {
    for (int t = q; t < 2 * NP * NPR; t += TPE) {
      const int D = t / (NP * NPR), ln = t / NPR % NP, pr = t % NPR, step = D ? RS : 1;
      const int base = el * ES + (D ? ln : ln * RS), ki = base + sa[pr] * step, kr = base + sb[pr] * step;
      double F[5];
      if (sfar[el][D][ln]) ecflux_log(node(ki, D), sp[6][ki], sp[7][ki], node(kr, D), sp[6][kr], sp[7][kr], cg, F);
      else ecflux_near(node(ki, D), node(kr, D), cg, T, F);
#pragma unroll
      for (int c = 0; c < 5; ++c) sF[el][D][ln][pr][c] = F[c];
    }
    if (face) {
      double F[5];
      face_flux(node(el * ES + fq, fD), sp[5][el * ES + fq], n, fD, fside, iface, mp.gamma, cg, F);
#pragma unroll
      for (int c = 0; c < 5; ++c) sG[el][fD][fside][fln][c] = F[c];
    }
  }
  __syncthreads();
  if (own) {
    const double rw = rcp_refined(T->w[0]);
    double acc[2][5];
#pragma unroll
    for (int D = 0; D < 2; ++D) {
      const int pos = D ? q / NP : q % NP, ln = D ? q % NP : q / NP;
#pragma unroll
      for (int c = 0; c < 5; ++c) acc[D][c] = 0.0;
#pragma unroll
      for (int side = 0; side < 2; ++side)
        if (pos == (side ? P : 0)) {
#pragma unroll
          for (int c = 0; c < 5; ++c) acc[D][c] = fma(side ? rw : -rw, sG[el][D][side][ln][c], acc[D][c]);
        }
#pragma unroll
      for (int r = 0; r < NP; ++r)
        if (r != pos) {
          const double* F = sF[el][D][ln][r < pos ? pair(r, pos) : pair(pos, r)];
#pragma unroll
          for (int c = 0; c < 5; ++c) acc[D][c] = fma(S[D][r], F[c], acc[D][c]);
        }
      const double sc = -2.0 * (D ? mp.rhy : mp.rhx);
#pragma unroll
      for (int c = 0; c < 5; ++c) acc[D][c] *= sc;
    }
    const double L[5] = {acc[0][0] + acc[1][0], acc[0][1] + acc[1][2], acc[0][2] + acc[1][1], acc[0][3] + acc[1][3],
                         acc[0][4] + acc[1][4]};
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      const double v = MODE == 0 ? L[c] : fma(cb * tau, L[c], Y[c]);
      bst(node_rsrc(out + c * KN, KN), no, v);
      sp[c][k] = v;
    }
  }
  if (MODE == 0) return;
  __syncthreads();
  stage_stats<P, BS, RS, ES>(sp[0], EB * ES, sp[5], e0, nel, stats, flag, T, mp.gamma);
}

template <int P, int MODE, int BS>
__global__ __launch_bounds__(BS) void k_hydro_stage_node(const double* __restrict__ Us, const double* __restrict__ Un,
                                                    double* __restrict__ out, double* __restrict__ stats,
                                                    int* __restrict__ flag, const HydroTab* __restrict__ T, MeshP mp,
                                                    double ca, double cb, double tau, int iface) {
  hydro_stage_node_body<P, MODE, BS>(Us, Un, out, stats, flag, T, mp, ca, cb, tau, iface, (long)blockIdx.x);
}

template <int P, int MODE, int BS>
__global__ __launch_bounds__(BS) void k_hydro_stage_node_rt(const hydro_stage_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const hydro_stage_args& a = A[r];
  hydro_stage_node_body<P, MODE, BS>(gl(a.Us), gl(a.Un), gl(a.out), gl(a.stats), gl(a.flag), gl(a.T), a.mp, a.ca, a.cb, a.tau, a.iface, (long)blockIdx.x - boff[r]);
}

template <int P>
__global__ __launch_bounds__(256) void k_elem_stats(const double* __restrict__ Uin, double* __restrict__ stats,
                                                    int* __restrict__ flag, const HydroTab* __restrict__ T, MeshP mp) {
  using C = Cfg<P>;
  constexpr int NP = C::NP, NN = C::NN, EB = C::EB;
  __shared__ double sv[7][EB * NN];  // rows 5 and 6: the sums
  const int tid = threadIdx.x, e0 = (int)blockIdx.x * EB;
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;
  const long KN = mp.K * NN;
  if (tid < nel * NN)
    for (int c = 0; c < 5; ++c) sv[c][tid] = Uin[c * KN + (long)e0 * NN + tid];
  __syncthreads();
  stage_stats<P, 256, NP, NN>(sv[0], EB * NN, sv[5], e0, nel, stats, flag, T, mp.gamma);
}

// pressure of a conserved state, and the size S_p that the pressure floor scales with
__device__ __forceinline__ double pres(const double* a, double g) {
  return (g - 1.0) * (a[4] - dot3(a[1], a[2], a[3], a[1], a[2], a[3]) / (2.0 * a[0]));
}
__device__ __forceinline__ double Sp(const double* a, double eps_r) {
  return fabs(a[4]) + dot3(a[1], a[2], a[3], a[1], a[2], a[3]) / (2.0 * fmax(a[0], eps_r));
}

// Pieces that the two forms of the stage map share.
// Cross-line amplitude shared by the components (eq. euler-oe-amplitude) from the statistics l of a row or column,
// rn its reciprocal weight sum
__device__ __forceinline__ double cross_amp(const double* __restrict__ l, const double* __restrict__ glob, double rn, double r4K) {
  double a = 0.0;
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    const double gm = glob[d * 3] * r4K, m = l[d * 3] * rn;
    const double dOm = fmax(glob[d * 3 + 2] - gm, gm - glob[d * 3 + 1]);
    a = fmax(a, fmax(fmax(l[d * 3 + 2] - m, m - l[d * 3 + 1]), 1e-6 * dOm));
  }
  return a;
}
// a component that is constant to roundoff (its nodal values agree to 2^10 ulps of its size, an exact test) does
// not count
__device__ __forceinline__ bool is_constant(const double* __restrict__ glob, int c) {
  const double gmn = glob[c * 3 + 1], gmx = glob[c * 3 + 2];
  return gmx - gmn <= 1024.0 * EPSM * fmax(fabs(gmx), fabs(gmn));
}
// damping rates (eq. euler-oe-rate) of an element with the averages a
template <int P>
__device__ __forceinline__ void damping_rates(const double a[5], double g, const MeshP& mp, double& lx, double& ly) {
  const double ir0 = 1.0 / a[0];
  const double pa = (g - 1.0) * fma(-0.5 * ir0, dot3(a[1], a[2], a[3], a[1], a[2], a[3]), a[4]);
  const double ck = sqrt(g * pa * ir0);
  lx = (2.0 * P + 1.0) * (fabs(a[1] * ir0) + ck) * mp.rhx;
  ly = (2.0 * P + 1.0) * (fabs(a[2] * ir0) + ck) * mp.rhy;
}
// D_l = exp(-s tau (lx sum_{r<=l} sigma_x,r + ly sum_{r<=l} sigma_y,r)) (eq. euler-oe-map)
__device__ __forceinline__ double shell_damping(int l, const double* sigx, const double* sigy, double lx, double ly, double st) {
  double sx = 0.0, sy = 0.0;
  for (int r = 0; r <= l; ++r) { sx += sigx[r]; sy += sigy[r]; }
  return l == 0 ? 1.0 : exp(-st * fma(lx, sx, ly * sy));
}
// the stage's node: conserved, and as the primitive copy for the magnetic substep (rho_o null: none)
__device__ __forceinline__ void store_node(const double U[5], unsigned no, long KN, double* __restrict__ Uout,
                                           double* __restrict__ rho_o, double* __restrict__ e_o, double* __restrict__ u_o) {
#pragma unroll
  for (int d = 0; d < 5; ++d) bst(node_rsrc(Uout + d * KN, KN), no, U[d]);
  if (rho_o) {
    const double r = U[0], ux = U[1] / r, uy = U[2] / r, uz = U[3] / r;
    bst(node_rsrc(rho_o, KN), no, r);
    bst(node_rsrc(u_o, KN), no, ux); bst(node_rsrc(u_o + KN, KN), no, uy); bst(node_rsrc(u_o + 2 * KN, KN), no, uz);
    bst(node_rsrc(e_o, KN), no, internal_energy(U[4], r, ux, uy, uz));
  }
}

// Tile of the hydro OE sensor: TX x TY elements and the ring around them, one thread per component and
// face.  The tile's (TX + 1) TY x faces run on the block's first half, its TX (TY + 1) y faces on the second
// (120 and 125 of 128 threads), so that a wave has one direction.
template <int P>
struct HS {
  static constexpr int NP = P + 1, NN = NP * NP, ES = NN | 1;  // odd element stride in LDS: no bank conflicts
  static constexpr int TX = 5, TY = 4, TE = TX * TY, BS = 256;
  static constexpr int NX = (TX + 1) * TY, NY = TX * (TY + 1);  // faces
  static constexpr int NS = TE + 2 * (TX + TY);                 // staged elements: the tile's, then the ring's
};

// Hydro OE sensor (eq. euler-oe-amplitude .. eq. euler-oe-map): the shell damping factors D_l (l = 0..p) of every
// element from the raw stage, Dfac[K][p+1].  Every face's jumps are formed once per tile, by a thread of
// its own from LDS; only the squared sums are exchanged.  Bound by VALU issue (1.3e8 instructions at
// 1024^2, N = 4) and its reads: 0.40 ms there (1.26 GB).
template <int P>
__device__ __forceinline__ void hydro_sensor_body(const double* __restrict__ Ust, const double* __restrict__ stats,
                                                  const double* __restrict__ lines, const double* __restrict__ glob,
                                                  double* __restrict__ Dfac, const int* __restrict__ flag,
                                                  const HydroTab* __restrict__ T, MeshP mp, double tau, double sH,
                                                  int blk) {
  using C = HS<P>;
  constexpr int NP = C::NP, NN = C::NN, ES = C::ES, TX = C::TX, TY = C::TY, TE = C::TE, BS = C::BS, NS = C::NS;
  constexpr int NX = C::NX, NY = C::NY;
  // su[c][staged element][ES]; then the faces' jumps sj[c][face][NP] (x faces first)
  constexpr int NU = 5 * NS * ES, NJ = 5 * (NX + NY) * NP;
  __shared__ double su[NU > NJ ? NU : NJ], ssg[TE][2 * NP], samp[2][TX], slam[2][TE];
  __shared__ int sel[NS];
  const int tid = threadIdx.x;
  int ty0, tx0;
  tile_of(blk, (mp.nx + TX - 1) / TX, (mp.ny + TY - 1) / TY, tx0, ty0);
  tx0 *= TX; ty0 *= TY;
  const int tw = mp.nx - tx0 < TX ? mp.nx - tx0 : TX, th = mp.ny - ty0 < TY ? mp.ny - ty0 : TY;  // tile in the mesh
  const long KN = mp.K * NN;
  const double g = mp.gamma;
  // the staged elements (ring: left, right column, bottom, top row), -1 where the mesh ends the tile early
  if (tid < NS) {
    const int s = tid;
    int x, y;
    bool in;
    if (s < TE) { y = s / TX; x = s - y * TX; in = x < tw && y < th; }
    else if (s < TE + 2 * TY) { const int h = s - TE; x = h < TY ? -1 : tw; y = h < TY ? h : h - TY; in = y < th; }
    else { const int h = s - TE - 2 * TY; y = h < TX ? -1 : th; x = h < TX ? h : h - TX; in = x < tw; }
    sel[s] = in ? wrap32(ty0 + y, mp.ny) * mp.nx + wrap32(tx0 + x, mp.nx) : -1;
  }
  __syncthreads();
  // their nodes, coalesced
  constexpr int NR = (NS * NN + BS - 1) / BS;
  double raw[NR][5];
  int slot[NR];
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int n = tid + m * BS, s = n / NN, q = n - s * NN;
    const int e = n < NS * NN ? sel[s] : -1;
    slot[m] = e < 0 ? -1 : s * ES + q;
    if (e >= 0)
#pragma unroll
      for (int d = 0; d < 5; ++d) raw[m][d] = bld(node_rsrc(Ust + d * KN, KN), ((unsigned)e * NN + q) * 8u);
  }
  if (flag && *flag) return;
  // cross-line amplitudes shared by the components (eq. euler-oe-amplitude): rows, then columns
  for (int t = tid; t < TY + TX; t += BS) {
    const int D = t < TY ? 0 : 1, i = D ? t - TY : t;
    if (i < (D ? tw : th)) {
      samp[D][i] = cross_amp(lines + (D ? mp.ny + tx0 + i : ty0 + i) * 15, glob, D ? mp.r4ny : mp.r4nx, mp.r4K);
    }
  }
  // wave speeds of the damping rate (eq. euler-oe-rate) from the element averages
  if (tid >= 64 && tid - 64 < TE) {
    const int en = tid - 64, x = en % TX, y = en / TX;
    if (x < tw && y < th) {
      const double* st = stats + (long)((ty0 + y) * mp.nx + tx0 + x) * 15;
      double a[5];
#pragma unroll
      for (int d = 0; d < 5; ++d) a[d] = 0.25 * st[3 * d];
      damping_rates<P>(a, g, mp, slam[0][en], slam[1][en]);
    }
  }
#pragma unroll
  for (int m = 0; m < NR; ++m)
    if (slot[m] >= 0)
#pragma unroll
      for (int d = 0; d < 5; ++d) su[d * NS * ES + slot[m]] = raw[m][d];
  __syncthreads();
  // the thread's face (x faces: fx counts the TX + 1 faces of a row) and component
  const int D = __builtin_amdgcn_readfirstlane(tid >= BS / 2 ? 1 : 0);
  const int t = tid - D * (BS / 2), nf = D ? NY : NX, c = t / nf, f = t - c * nf;
  const int fx = D ? f % TX : f % (TX + 1), fy = D ? f / TX : f / (TX + 1);
  const bool act = c < 5 && (D ? fx < tw && fy <= th : fx <= tw && fy < th);
  double J[NP];
  if (act) {
    const double* S = su + c * NS * ES;
    if (D == 0)
      face_jumps<P, 0>(S + (fx == 0 ? TE + fy : fy * TX + fx - 1) * ES, S + (fx == tw ? TE + TY + fy : fy * TX + fx) * ES, T, J);
    else
      face_jumps<P, 1>(S + (fy == 0 ? TE + 2 * TY + fx : (fy - 1) * TX + fx) * ES,
                       S + (fy == th ? TE + 2 * TY + TX + fx : fy * TX + fx) * ES, T, J);
  }
  __syncthreads();
  if (act) {
    const bool cst = is_constant(glob, c);
    double* o = su + (c * (NX + NY) + (D ? NX + f : f)) * NP;
#pragma unroll
    for (int r = 0; r < NP; ++r) o[r] = cst ? 0.0 : J[r];
  }
  __syncthreads();
  // sigma (eq. euler-oe-sigma): the two faces' jumps, maximum over the components, against the shared amplitude
  for (int k = tid; k < TE * 2 * NP; k += BS) {
    const int r = k % NP, d = (k / NP) & 1, en = k / (2 * NP), x = en % TX, y = en / TX;
    if (x < tw && y < th) {
      const int f0 = d ? NX + y * TX + x : y * (TX + 1) + x, f1 = f0 + (d ? TX : 1);
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < 5; ++q)
        s = fmax(s, su[(q * (NX + NY) + f0) * NP + r] + su[(q * (NX + NY) + f1) * NP + r]);
      const double A = samp[d][d ? x : y];
      ssg[en][d * NP + r] = A > 0.0 ? T->fr[r] * s / A : 0.0;
    }
  }
  __syncthreads();
  for (int k = tid; k < TE * NP; k += BS) {
    const int l = k % NP, en = k / NP, x = en % TX, y = en / TX;
    if (x < tw && y < th)
      Dfac[(long)((ty0 + y) * mp.nx + tx0 + x) * NP + l] =
          shell_damping(l, ssg[en], ssg[en] + NP, slam[0][en], slam[1][en], sH * tau);
  }
}

template <int P>
__global__ __launch_bounds__(HS<P>::BS) void k_hydro_sensor(const double* __restrict__ Ust, const double* __restrict__ stats,
                                                  const double* __restrict__ lines, const double* __restrict__ glob,
                                                  double* __restrict__ Dfac, const int* __restrict__ flag,
                                                  const HydroTab* __restrict__ T, MeshP mp, double tau, double sH) {
  hydro_sensor_body<P>(Ust, stats, lines, glob, Dfac, flag, T, mp, tau, sH, (int)xcd_block());
}

struct hydro_sensor_args {
  const double* Ust;
  const double* stats;
  const double* lines;
  const double* glob;
  double* Dfac;
  const int* flag;
  const HydroTab* T;
  MeshP mp;
  double tau;
  double sH;
};

template <int P>
__global__ __launch_bounds__(HS<P>::BS) void k_hydro_sensor_rt(const hydro_sensor_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const hydro_sensor_args& a = A[r];
  hydro_sensor_body<P>(gl(a.Ust), gl(a.stats), gl(a.lines), gl(a.glob), gl(a.Dfac), gl(a.flag), gl(a.T), a.mp, a.tau, a.sH, (int)blockIdx.x - boff[r]);
}

// Discrete Legendre transform of a grid line and its inverse.  On the symmetric GLL nodes
// Tf[a][k] = (-1)^a Tf[a][p-k] and V[k][a] = (-1)^a V[p-k][a], bit for bit in the tables, so the line's even
// and odd parts are transformed.
template <int P>
__device__ __forceinline__ void legendre_fwd(const double* v, double* m, const HydroTab* __restrict__ T) {
  constexpr int NP = P + 1, H = NP / 2;
  double e[H + 1], o[H + 1];
#pragma unroll
  for (int k = 0; k < H; ++k) { e[k] = v[k] + v[P - k]; o[k] = v[k] - v[P - k]; }
  if (NP % 2) e[H] = v[H];
#pragma unroll
  for (int a = 0; a < NP; ++a) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < (a % 2 ? H : NP - H); ++k) s = fma(T->Tf[a][k], a % 2 ? o[k] : e[k], s);
    m[a] = s;
  }
}
template <int P>
__device__ __forceinline__ void legendre_inv(const double* m, double* v, const HydroTab* __restrict__ T) {
  constexpr int NP = P + 1, H = NP / 2;
#pragma unroll
  for (int k = 0; k < NP - H; ++k) {
    double e = 0.0, o = 0.0;
#pragma unroll
    for (int a = 0; a < NP; a += 2) e = fma(T->V[k][a], m[a], e);
    if (k < H)
#pragma unroll
      for (int a = 1; a < NP; a += 2) o = fma(T->V[k][a], m[a], o);
    v[k] = e + o;
    if (k < H) v[P - k] = e - o;
  }
}

// Block of the stage map: EB consecutive elements, one thread per (component, element).
template <int P>
struct OM {
  static constexpr int NP = P + 1, NN = NP * NP, ES = NN | 1;  // odd element stride in LDS: no bank conflicts
  static constexpr int EB = 24, BS = 128;                      // 120 of 128 threads
};

// P = P_PP o P_OE on a raw stage (eq. euler-oe-map, eq. euler-pp-density, eq. euler-pp-pressure) with the damping
// factors Dfac of the sensor.  A thread holds one component of an element in registers: the modal transforms
// and the damping are straight-line code with the 1D tables as scalars.  The
// element statistics of the raw stage (always formed before this map) give the element averages: the map
// keeps each element's mean, the (0, 0) Legendre mode.  Bound by HBM: 2.4 GB in 0.46 ms at 1024^2, N = 4.
// All modes are transformed, also where nothing is damped: D_p U plus the others' (D_l - D_p) takes the same time, and with it
// ||div B|| at the end of the rotor run, a quantity of round-off alone, comes out 20 % below the published value that
// its test holds within 5 %.
//
// One kernel for sensor and map, with a thread per element line and component that formed its neighbours'
// traces too, was bound by VALU issue and LDS alike (4.5e8 VALU instructions, 4.5e8 LDS cycles): 1.23 ms at
// 1024^2, N = 4 against 0.86 for the two, 0.324 against 0.152 ms at 512^2, N = 3 (20 line tasks on an element's
// 16 threads), 38 against 27 us at 256^2, N = 2, 70 against 57 us at 241 x 137, N = 5.  One kernel with a thread
// per component and element that exchanges its traces through LDS took 1.18 ms: its 16 barriers and 160
// registers leave two blocks on a CU.
template <int P>
__device__ __forceinline__ void hydro_oe_pp_body(const double* __restrict__ Ust, double* __restrict__ Uout,
                                                     const double* __restrict__ stats, const double* __restrict__ Dfac,
                                                     uint8_t* __restrict__ flags,
                                                     unsigned long long* __restrict__ counts,
                                                     const int* __restrict__ flag, const HydroTab* __restrict__ T,
                                                     MeshP mp, int do_oe, int do_pp,
                                                     double* __restrict__ rho_o, double* __restrict__ e_o,
                                                     double* __restrict__ u_o, long blk) {
  using C = OM<P>;
  constexpr int NP = C::NP, NN = C::NN, ES = C::ES, EB = C::EB, BS = C::BS;
  __shared__ double su[5][EB * ES];
  __shared__ double sa[5][EB], sred[2][5][EB], sth[2][EB], srmin[EB];
  const int tid = threadIdx.x, c = tid / EB, el = tid - c * EB;
  const int e0 = (int)(blk * EB);
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;
  const bool act = c < 5 && el < nel;
  const long KN = mp.K * NN;
  const int e = e0 + el;
  const double g = mp.gamma;
  constexpr int NR = (EB * NN + BS - 1) / BS;
  {
    double raw[NR][5];
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = tid + m * BS;
      if (n < nel * NN)
#pragma unroll
        for (int d = 0; d < 5; ++d) raw[m][d] = bld(node_rsrc(Ust + d * KN, KN), ((unsigned)e0 * NN + n) * 8u);
    }
    if (flag && *flag) return;
    if (act) {
      sa[c][el] = 0.25 * stats[((long)e * 5 + c) * 3];
      if (c == 0 && !do_oe) srmin[el] = stats[(long)e * 15 + 1];  // raw-stage density minimum
    }
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = tid + m * BS;
      if (n < nel * NN)
#pragma unroll
        for (int d = 0; d < 5; ++d) su[d][n / NN * ES + n % NN] = raw[m][d];
    }
  }
  __syncthreads();
  if (do_oe) {
    if (act) {
      double* const mine = su[c] + el * ES;
      double f[NP];
#pragma unroll
      for (int l = 0; l < NP; ++l) f[l] = Dfac[(long)e * NP + l];
      double w[NP][NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        double v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) v[i] = mine[j * NP + i];
        legendre_fwd<P>(v, w[j], T);
      }
#pragma unroll
      for (int a = 0; a < NP; ++a) {
        double col[NP], m[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) col[j] = w[j][a];
        legendre_fwd<P>(col, m, T);
#pragma unroll
        for (int b = 0; b < NP; ++b) m[b] *= f[a > b ? a : b];
        legendre_inv<P>(m, col, T);
#pragma unroll
        for (int j = 0; j < NP; ++j) w[j][a] = col[j];
      }
      double mn = DBL_MAX;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        double o[NP];
        legendre_inv<P>(w[j], o, T);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          mine[j * NP + i] = o[i];
          mn = fmin(mn, o[i]);
        }
      }
      if (c == 0) srmin[el] = mn;
    }
    __syncthreads();
  }
  // positivity scaling: S_p and the pressure minimum over the nodes by the element's five threads, the
  // two factors by one of them, applied as the nodes are written
  const double eps_r = 64.0 * EPSM;
  if (do_pp) {
    double a0 = 0.0, thr = 1.0;
    bool collapse = false;
    if (act) {
      a0 = sa[0][el];
      collapse = !(a0 > eps_r);
      const double rmin = srmin[el];
      if (!collapse && rmin < eps_r) thr = fmin(1.0, fmax(0.0, (a0 - eps_r) / (a0 - rmin)));
      double S = 0.0, pm = DBL_MAX;
#pragma unroll
      for (int k = 0; k < (NN + 4) / 5; ++k) {
        const int q = c + 5 * k;
        if (q < NN) {
          double U[5];
#pragma unroll
          for (int d = 0; d < 5; ++d) U[d] = su[d][el * ES + q];
          if (thr != 1.0) U[0] = a0 + thr * (U[0] - a0);
          S = fmax(S, Sp(U, eps_r));
          pm = fmin(pm, pres(U, g));
        }
      }
      sred[0][c][el] = S;
      sred[1][c][el] = pm;
    }
    __syncthreads();
    if (act && c == 0) {
      double a[5], thp = 1.0;
      int f = 0;
#pragma unroll
      for (int d = 0; d < 5; ++d) a[d] = sa[d][el];
      if (collapse) {
        f = 4;
      } else {
        f = srmin[el] < eps_r ? 1 : 0;
        double S = Sp(a, eps_r), pmin = DBL_MAX;
#pragma unroll
        for (int d = 0; d < 5; ++d) { S = fmax(S, sred[0][d][el]); pmin = fmin(pmin, sred[1][d][el]); }
        const double eps_p = fmax(64.0 * EPSM, 8192.0 * EPSM * S);
        const double pb = pres(a, g);
        if (pb <= eps_p) {
          f |= 4;
        } else if (pmin < eps_p) {
          thp = fmin(1.0, fmax(0.0, (pb - eps_p) / (pb - pmin)));
          f |= 2;
        }
      }
      sth[0][el] = thr;
      sth[1][el] = (f & 4) ? -1.0 : thp;  // -1: collapsed to the average
      if (flags) flags[e] = (uint8_t)f;
      if (counts && f) {
        if (f & 1) atomicAdd(&counts[0], 1ull);
        if (f & 2) atomicAdd(&counts[1], 1ull);
        if (f & 4) atomicAdd(&counts[2], 1ull);
      }
    }
    __syncthreads();
  } else if (act && c == 0 && flags) {
    flags[e] = 0;
  }
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const int n = tid + m * BS;
    if (n >= nel * NN) continue;
    const unsigned no = ((unsigned)e0 * NN + n) * 8u;
    const int en = n / NN, k = en * ES + n % NN;
    double U[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) U[d] = su[d][k];
    if (do_pp) {
      const double thr = sth[0][en], thp = sth[1][en];
      if (thr != 1.0) U[0] = sa[0][en] + thr * (U[0] - sa[0][en]);
      if (thp != 1.0) {
#pragma unroll
        for (int d = 0; d < 5; ++d) U[d] = thp < 0.0 ? sa[d][en] : sa[d][en] + thp * (U[d] - sa[d][en]);
      }
    }
    store_node(U, no, KN, Uout, rho_o, e_o, u_o);
  }
}

template <int P>
__global__ __launch_bounds__(OM<P>::BS) void k_hydro_oe_pp(const double* __restrict__ Ust, double* __restrict__ Uout,
                                                     const double* __restrict__ stats, const double* __restrict__ Dfac,
                                                     uint8_t* __restrict__ flags,
                                                     unsigned long long* __restrict__ counts,
                                                     const int* __restrict__ flag, const HydroTab* __restrict__ T,
                                                     MeshP mp, int do_oe, int do_pp,
                                                     double* __restrict__ rho_o, double* __restrict__ e_o,
                                                     double* __restrict__ u_o) {
  hydro_oe_pp_body<P>(Ust, Uout, stats, Dfac, flags, counts, flag, T, mp, do_oe, do_pp, rho_o, e_o, u_o, xcd_block());
}

struct hydro_oe_pp_args {
  const double* Ust;
  double* Uout;
  const double* stats;
  const double* Dfac;
  uint8_t* flags;
  unsigned long long* counts;
  const int* flag;
  const HydroTab* T;
  MeshP mp;
  int do_oe;
  int do_pp;
  double* rho_o;
  double* e_o;
  double* u_o;
};

template <int P>
__global__ __launch_bounds__(OM<P>::BS) void k_hydro_oe_pp_rt(const hydro_oe_pp_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const hydro_oe_pp_args& a = A[r];
  hydro_oe_pp_body<P>(gl(a.Ust), gl(a.Uout), gl(a.stats), gl(a.Dfac), gl(a.flags), gl(a.counts), gl(a.flag), gl(a.T), a.mp, a.do_oe, a.do_pp, gl(a.rho_o), gl(a.e_o), gl(a.u_o), (long)blockIdx.x - boff[r]);
}

// The whole stage map in one launch, for small and for one element wide meshes (see one_launch_map): the derivative jumps
// and the modal transforms run as line tasks, task (c, line) holding one grid line of component c in registers (five
// tasks per line index, EB elements per block); an element forms its neighbours' traces again.  Same arithmetic
// as the two kernels above, whose threads work through an element and whose launch of its own counts here: at 24^2, N = 4
// 8.9 against 6.6 + 6.6 us, N = 6 12.2 against 9.8 + 11 us.
constexpr int ML_BS = 128;
template <int P>
__device__ __forceinline__ void hydro_map_lines_body(const double* __restrict__ Ust, double* __restrict__ Uout,
                                                     const double* __restrict__ stats, const double* __restrict__ lines,
                                                     const double* __restrict__ glob, uint8_t* __restrict__ flags,
                                                     unsigned long long* __restrict__ counts,
                                                     const int* __restrict__ flag, const HydroTab* __restrict__ T,
                                                     MeshP mp, double tau, double sH, int do_pp,
                                                     double* __restrict__ rho_o, double* __restrict__ e_o,
                                                     double* __restrict__ u_o, long blk) {
  using C = Cfg<P, ML_BS>;
  constexpr int NP = C::NP, NN = C::NN, EB = C::EB, NL = 5 * NP;
  __shared__ double su[5][EB * NN], st[10][EB * NN];
  __shared__ double ssig[EB][2][NP], ssg[EB][5][NP], sD[EB][NP], samp[EB][2], srow[EB][3][NP];
  if (flag && *flag) return;
  const int tid = threadIdx.x;
  const int el = tid / NN, q = tid - el * NN;
  const long e = blk * EB + el;
  const bool act = tid < C::NT && e < mp.K;
  const long KN = mp.K * NN;
  const unsigned no = ((unsigned)e * NN + q) * 8u;  // the node's byte offset in a component array
  const double g = mp.gamma;
  int ex, ey;
  elem_xy32(mp, act ? (int)e : 0, ex, ey);
  // grid line ln of direction D (D = 0: row, index along x; D = 1: column), position k on it
  auto nodeof = [](int D, int ln, int k) { return D == 0 ? ln * NP + k : k * NP + ln; };
  double U[5], a[5], rmin = 1.0;
  // the four neighbours' nodes (x minus, x plus, y minus, y plus) are loaded into registers up
  // front with the element's own, so that their latency overlaps the amplitude and x phases; they
  // go to LDS when their direction comes
  double nb[4][5];
  if (act) {
    const int nbe[4] = {ey * mp.nx + wrap32(ex - 1, mp.nx), ey * mp.nx + wrap32(ex + 1, mp.nx),
                        wrap32(ey - 1, mp.ny) * mp.nx + ex, wrap32(ey + 1, mp.ny) * mp.nx + ex};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const unsigned on = ((unsigned)nbe[s] * NN + q) * 8u;
#pragma unroll
      for (int c = 0; c < 5; ++c) nb[s][c] = bld(node_rsrc(Ust + c * KN, KN), on);
    }
  }
  if (act) {
#pragma unroll
    for (int c = 0; c < 5; ++c) { U[c] = bld(node_rsrc(Ust + c * KN, KN), no); su[c][tid] = U[c]; }
#pragma unroll
    for (int c = 0; c < 5; ++c) a[c] = 0.25 * stats[(e * 5 + c) * 3];
  }
  __syncthreads();
  if (act && q < 2) samp[el][q] = cross_amp(lines + (q ? mp.ny + ex : ey) * 15, glob, q ? mp.r4ny : mp.r4nx, mp.r4K);
#pragma unroll
  for (int D = 0; D < 2; ++D) {
    // neighbours across the two faces normal to direction D, staged in st rows 0..9
    // (row c: minus-side neighbour, row 5 + c: plus-side neighbour)
    if (act) {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        st[c][tid] = nb[2 * D][c];
        st[5 + c][tid] = nb[2 * D + 1][c];
      }
    }
    __syncthreads();
    // jumps of the derivatives (see face_jumps) of line ln of component c at the element's two faces, into the
    // task's own staged slots (order r at position r of the line)
    for (int t = q; act && t < NL; t += NN) {
      const int ln = t / 5, c = t - ln * 5;  // component fastest (fewer LDS bank conflicts)
      double own[NP], mn[NP], pl[NP];
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const int n = el * NN + nodeof(D, ln, k);
        own[k] = su[c][n]; mn[k] = st[c][n]; pl[k] = st[5 + c][n];
      }
#pragma unroll
      for (int r = 0; r < NP; ++r) {
        const int n = el * NN + nodeof(D, ln, r);
        st[c][n] = line_jump<P>(mn, own, r, T);
        st[5 + c][n] = line_jump<P>(own, pl, r, T);
      }
    }
    __syncthreads();
    // their norms over the lines, both faces together: task (r, c)
    for (int t = q; act && t < NL; t += NN) {
      const int r = t / 5, c = t - r * 5;
      double Jm = 0.0, Jp = 0.0;
#pragma unroll
      for (int l = 0; l < NP; ++l) {
        const int n = el * NN + nodeof(D, l, r);
        Jm = fma(0.5 * T->w[l] * st[c][n], st[c][n], Jm);
        Jp = fma(0.5 * T->w[l] * st[5 + c][n], st[5 + c][n], Jp);
      }
      ssg[el][c][r] = is_constant(glob, c) ? 0.0 : sqrt(Jm) + sqrt(Jp);
    }
    __syncthreads();
    if (act && q < NP) {  // sigma (eq. euler-oe-sigma): maximum over the components, against the shared amplitude
      double sg = 0.0;
#pragma unroll
      for (int c = 0; c < 5; ++c) sg = fmax(sg, ssg[el][c][q]);
      const double A = samp[el][D];
      ssig[el][D][q] = A > 0.0 ? T->fr[q] * sg / A : 0.0;
    }
  }
  // modal damping with line tasks: x transform of each row, then per column the y transform,
  // the shell factors and the inverse y transform, then the inverse x transform of each row
  for (int t = q; act && t < NL; t += NN) {
    const int ln = t / 5, c = t - ln * 5;  // component fastest (fewer LDS bank conflicts)
    double v[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = su[c][el * NN + ln * NP + k];
    double m[NP];
    legendre_fwd<P>(v, m, T);
#pragma unroll
    for (int k = 0; k < NP; ++k) st[c][el * NN + ln * NP + k] = m[k];  // [row][x mode]
  }
  __syncthreads();
  if (act && q < NP) {
    double lx, ly;
    damping_rates<P>(a, g, mp, lx, ly);
    sD[el][q] = shell_damping(q, ssig[el][0], ssig[el][1], lx, ly, sH * tau);
  }
  __syncthreads();
  for (int t = q; act && t < NL; t += NN) {
    const int aa = t / 5, c = t - aa * 5;
    double v[NP], m[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = st[c][el * NN + k * NP + aa];
    legendre_fwd<P>(v, m, T);
#pragma unroll
    for (int b = 0; b < NP; ++b) m[b] *= sD[el][aa > b ? aa : b];
    legendre_inv<P>(m, v, T);
#pragma unroll
    for (int k = 0; k < NP; ++k) st[c][el * NN + k * NP + aa] = v[k];
  }
  __syncthreads();
  for (int t = q; act && t < NL; t += NN) {
    const int ln = t / 5, c = t - ln * 5;
    double m[NP], v[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) m[k] = st[c][el * NN + ln * NP + k];
    legendre_inv<P>(m, v, T);
    double mn = DBL_MAX;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      su[c][el * NN + ln * NP + k] = v[k];
      mn = fmin(mn, v[k]);
    }
    if (c == 0) srow[el][0][ln] = mn;  // row minimum of the damped density
  }
  __syncthreads();
  if (act) {
#pragma unroll
    for (int c = 0; c < 5; ++c) U[c] = su[c][tid];
    rmin = DBL_MAX;
#pragma unroll
    for (int l = 0; l < NP; ++l) rmin = fmin(rmin, srow[el][0][l]);
  }
  uint8_t f = 0;
  if (do_pp) {
    // positivity scaling: the S_p and pressure extrema are reduced per row (NP tasks per
    // element), then over the rows by every thread
    const double eps_r = 64.0 * EPSM;
    const bool collapse_r = !(a[0] > eps_r);
    double thr = 1.0;
    if (act && !collapse_r && rmin < eps_r) {
      thr = fmin(1.0, fmax(0.0, (a[0] - eps_r) / (a[0] - rmin)));
      f |= 1;
      if (thr != 1.0) U[0] = a[0] + thr * (U[0] - a[0]);  // density-limited state of this node
    }
    if (act) {
      st[0][tid] = Sp(U, eps_r);
      st[1][tid] = pres(U, g);
    }
    __syncthreads();
    for (int t = q; act && t < NP; t += NN) {
      double S = 0.0, pm = DBL_MAX;
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        S = fmax(S, st[0][el * NN + t * NP + k]);
        pm = fmin(pm, st[1][el * NN + t * NP + k]);
      }
      srow[el][1][t] = S;
      srow[el][2][t] = pm;
    }
    __syncthreads();
    if (act && !collapse_r) {
      double S = Sp(a, eps_r), pmin = DBL_MAX;
#pragma unroll
      for (int l = 0; l < NP; ++l) { S = fmax(S, srow[el][1][l]); pmin = fmin(pmin, srow[el][2][l]); }
      const double eps_p = fmax(64.0 * EPSM, 8192.0 * EPSM * S);
      const double pb = pres(a, g);
      if (pb <= eps_p) {
        f |= 4;
#pragma unroll
        for (int c = 0; c < 5; ++c) U[c] = a[c];
      } else if (pmin < eps_p) {
        const double thp = fmin(1.0, fmax(0.0, (pb - eps_p) / (pb - pmin)));
        f |= 2;
        if (thp != 1.0)
#pragma unroll
          for (int c = 0; c < 5; ++c) U[c] = a[c] + thp * (U[c] - a[c]);
      }
    } else if (act && collapse_r) {
      f = 4;
#pragma unroll
      for (int c = 0; c < 5; ++c) U[c] = a[c];
    }
  }
  if (act) {
    store_node(U, no, KN, Uout, rho_o, e_o, u_o);
    if (q == 0) {
      if (flags) flags[e] = f;
      if (counts && f) {
        if (f & 1) atomicAdd(&counts[0], 1ull);
        if (f & 2) atomicAdd(&counts[1], 1ull);
        if (f & 4) atomicAdd(&counts[2], 1ull);
      }
    }
  }
}

template <int P>
__global__ __launch_bounds__(ML_BS) void k_hydro_map_lines(const double* __restrict__ Ust, double* __restrict__ Uout,
                                                     const double* __restrict__ stats, const double* __restrict__ lines,
                                                     const double* __restrict__ glob, uint8_t* __restrict__ flags,
                                                     unsigned long long* __restrict__ counts,
                                                     const int* __restrict__ flag, const HydroTab* __restrict__ T,
                                                     MeshP mp, double tau, double sH, int do_pp,
                                                     double* __restrict__ rho_o, double* __restrict__ e_o,
                                                     double* __restrict__ u_o) {
  hydro_map_lines_body<P>(Ust, Uout, stats, lines, glob, flags, counts, flag, T, mp, tau, sH, do_pp, rho_o, e_o, u_o, xcd_block());
}

struct hydro_map_lines_args {
  const double* Ust;
  double* Uout;
  const double* stats;
  const double* lines;
  const double* glob;
  uint8_t* flags;
  unsigned long long* counts;
  const int* flag;
  const HydroTab* T;
  MeshP mp;
  double tau;
  double sH;
  int do_pp;
  double* rho_o;
  double* e_o;
  double* u_o;
};

template <int P>
__global__ __launch_bounds__(ML_BS) void k_hydro_map_lines_rt(const hydro_map_lines_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const hydro_map_lines_args& a = A[r];
  hydro_map_lines_body<P>(gl(a.Ust), gl(a.Uout), gl(a.stats), gl(a.lines), gl(a.glob), gl(a.flags), gl(a.counts), gl(a.flag), gl(a.T), a.mp, a.tau, a.sH, a.do_pp, gl(a.rho_o), gl(a.e_o), gl(a.u_o), (long)blockIdx.x - boff[r]);
}

// Connectivity export: nbr[K][4] (left, right, bottom, top neighbour) and the face map
// fmap[K][4][p+1] (the neighbour node e' (p+1)^2 + q' matched to each own face node), formed with the
// same face_match the stage kernel uses.  One thread per (element, face).
template <int P>
__global__ __launch_bounds__(256) void k_face_map(int32_t* __restrict__ nbr, int32_t* __restrict__ fmap, MeshP mp) {
  constexpr int NP = P + 1, NN = NP * NP;
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 4 * mp.K) return;
  const long e = t >> 2;
  const int f = (int)(t & 3), D = f >> 1, side = f & 1;
  int ex, ey;
  elem_xy32(mp, (int)e, ex, ey);
  int en = 0;
  for (int line = 0; line < NP; ++line) {
    int qo, qn;
    face_match<P>(mp, ex, ey, D, side, line, en, qo, qn);
    if (fmap) fmap[t * NP + line] = en * NN + qn;
  }
  nbr[t] = en;
}

// Entry copy of a conservative state with the admissibility test of every node: all five values
// finite, rho > 0 and p > 0 (the admissible set of section "Conservative ideal MHD").  A failing node
// sets bit 1 of flag[1].  One thread per node.
__device__ __forceinline__ void snap_check_node(const double* __restrict__ U, double* __restrict__ snap, long KN,
                                                double g, int* __restrict__ flag, long n) {
  double v[5];
  bool fin = true;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    v[c] = U[c * KN + n];
    snap[c * KN + n] = v[c];
    fin = fin && fabs(v[c]) <= DBL_MAX;
  }
  const double p = (g - 1.0) * (v[4] - (v[1] * v[1] + v[2] * v[2] + v[3] * v[3]) / (2.0 * v[0]));
  if (!fin || !(v[0] > 0.0) || !(p > 0.0)) atomicOr(flag + 1, 2);
}

// the same of an entry copy of the magnetic grids (finiteness), entry k of B_x, B_y and B_z
__device__ __forceinline__ void snap_check_B(const double* __restrict__ Bx, const double* __restrict__ By,
                                             const double* __restrict__ Bz, double* __restrict__ snap, long G,
                                             int* __restrict__ flag, long k) {
  const double x = Bx[k], y = By[k], z = Bz[k];
  snap[k] = x; snap[G + k] = y; snap[2 * G + k] = z;
  if (!(fabs(x) <= DBL_MAX && fabs(y) <= DBL_MAX && fabs(z) <= DBL_MAX)) atomicOr(flag + 1, 2);
}

// The entry copy in one launch (on small meshes launches cost more than the copies: 3 us saved per launch).
// G = 0: no magnetic grids.
__global__ __launch_bounds__(256) void k_snap_check(const double* __restrict__ U, double* __restrict__ snapU, long KN, double g,
                                                    const double* __restrict__ Bx, const double* __restrict__ By,
                                                    const double* __restrict__ Bz, double* __restrict__ snapB, long G,
                                                    int* __restrict__ flag) {
  const long k0 = (long)blockIdx.x * blockDim.x + threadIdx.x, dk = (long)gridDim.x * blockDim.x;
  for (long n = k0; n < KN; n += dk) snap_check_node(U, snapU, KN, g, flag, n);
  for (long k = k0; k < G; k += dk) snap_check_B(Bx, By, Bz, snapB, G, flag, k);
}

}  // namespace

// Row / column reduction of per-element statistics [K][nc][3] (sum, min, max), nc <= 5, fixed
// order.  Blocks 0..ny-1 reduce one element row each: thread t takes elements t, t+256, ... of
// the row and reads each element's nc*3 values as one contiguous record.  Blocks ny.. reduce
// LRC adjacent element columns each: thread (column j, phase p) takes rows p, p+LRP, ... of
// column j, so a wave reads adjacent elements of one row.  Partial results are combined in LDS
// by a fixed tree.
constexpr int LRC = 8, LRP = 256 / LRC;

// A row reduces its first rx elements and a column its first ry (the whole mesh on a periodic
// domain; the box of a mirror-walled mesh, whose other elements are mirror images: every row's and
// column's statistics are then those of the box's own, up to the sign of an odd field).
template <int NC>
__device__ __forceinline__ void line_reduce_body(const double* __restrict__ stats, double* __restrict__ lines,
                                                     int nx, int ny, int rx, int ry, const int* __restrict__ flag,
                                                     long blk) {
  constexpr int nc = NC;  // components per element record (compile-time, so that no load waits on a branch)
  __shared__ double red[15][256];
  if (flag && *flag) return;
  const int b = blk, t = threadIdx.x;
  const int nv = nc * 3;
  double v[15];
#pragma unroll
  for (int k = 0; k < 15; ++k) v[k] = (k % 3 == 0) ? 0.0 : (k % 3 == 1 ? DBL_MAX : -DBL_MAX);
  auto take = [&](long e) {
    const double* st = stats + e * nv;
#pragma unroll
    for (int c = 0; c < 5; ++c)
      if (c < nc) {
        v[3 * c] += st[3 * c];
        v[3 * c + 1] = fmin(v[3 * c + 1], st[3 * c + 1]);
        v[3 * c + 2] = fmax(v[3 * c + 2], st[3 * c + 2]);
      }
  };
  // (unrolled by 4 so that four records' loads are in flight at once; the accumulation order, and so
  // every result bit, is that of the plain loop)
  if (b < ny) {
#pragma unroll 4
    for (int k = t; k < rx; k += 256) take((long)b * nx + k);
  } else {
    const int col = (b - ny) * LRC + t % LRC, ph = t / LRC;
    if (col < nx)
#pragma unroll 4
      for (int r = ph; r < ry; r += LRP) take((long)r * nx + col);
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) red[k][t] = v[k];
  __syncthreads();
  // rows: tree over all 256 threads; columns: tree over the LRP phases of each column
  const int lo = b < ny ? 1 : LRC;
  for (int w = 128; w >= lo; w >>= 1) {
    if (t < w)
      for (int c = 0; c < nc; ++c) {
        red[3 * c][t] += red[3 * c][t + w];
        red[3 * c + 1][t] = fmin(red[3 * c + 1][t], red[3 * c + 1][t + w]);
        red[3 * c + 2][t] = fmax(red[3 * c + 2][t], red[3 * c + 2][t + w]);
      }
    __syncthreads();
  }
  if (b < ny) {
    if (t < nv) lines[(long)b * nv + t] = red[t][0];
  } else if (t < LRC * nv) {
    const int j = t % LRC, k = t / LRC, col = (b - ny) * LRC + j;
    if (col < nx) lines[((long)ny + col) * nv + k] = red[k][j];
  }
}

template <int NC>
__global__ __launch_bounds__(256) void k_line_reduce(const double* __restrict__ stats, double* __restrict__ lines,
                                                     int nx, int ny, int rx, int ry, const int* __restrict__ flag) {
  line_reduce_body<NC>(stats, lines, nx, ny, rx, ry, flag, (long)blockIdx.x);
}

struct line_reduce_args {
  const double* stats;
  double* lines;
  int nx;
  int ny;
  int rx;
  int ry;
  const int* flag;
};

template <int NC>
__global__ __launch_bounds__(256) void k_line_reduce_rt(const line_reduce_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const line_reduce_args& a = A[r];
  line_reduce_body<NC>(gl(a.stats), gl(a.lines), a.nx, a.ny, a.rx, a.ry, gl(a.flag), (long)blockIdx.x - boff[r]);
}

// Global reduction of the first `n` line results (the rows of the periodic mesh or of the box) into glob[nc][3]: all NC components in
// one tree (each component's accumulation order is that of its own tree), so the block passes
// eight barriers instead of eight per component.
template <int NC>
__device__ __forceinline__ void global_reduce_body(const double* __restrict__ lines, double* __restrict__ glob,
                                                       int n, const int* __restrict__ flag, long blk) {
  __shared__ double red[3 * NC][256];
  if (flag && *flag) return;
  const int t = threadIdx.x;
  double v[3 * NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) { v[3 * c] = 0.0; v[3 * c + 1] = DBL_MAX; v[3 * c + 2] = -DBL_MAX; }
  for (int k = t; k < n; k += 256) {
    const double* st = lines + (long)k * NC * 3;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      v[3 * c] += st[3 * c];
      v[3 * c + 1] = fmin(v[3 * c + 1], st[3 * c + 1]);
      v[3 * c + 2] = fmax(v[3 * c + 2], st[3 * c + 2]);
    }
  }
#pragma unroll
  for (int x = 0; x < 3 * NC; ++x) red[x][t] = v[x];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        red[3 * c][t] += red[3 * c][t + w];
        red[3 * c + 1][t] = fmin(red[3 * c + 1][t], red[3 * c + 1][t + w]);
        red[3 * c + 2][t] = fmax(red[3 * c + 2][t], red[3 * c + 2][t + w]);
      }
    __syncthreads();
  }
  if (t < 3 * NC) glob[t] = red[t][0];
}

template <int NC>
__global__ __launch_bounds__(256) void k_global_reduce(const double* __restrict__ lines, double* __restrict__ glob,
                                                       int n, const int* __restrict__ flag) {
  global_reduce_body<NC>(lines, glob, n, flag, (long)blockIdx.x);
}

struct global_reduce_args {
  const double* lines;
  double* glob;
  int n;
  const int* flag;
};

template <int NC>
__global__ __launch_bounds__(256) void k_global_reduce_rt(const global_reduce_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const global_reduce_args& a = A[r];
  global_reduce_body<NC>(gl(a.lines), gl(a.glob), a.n, gl(a.flag), (long)blockIdx.x - boff[r]);
}

// argument structs of the small and flat kernels for run-table launches
struct reset_args {
  int* flag;
  unsigned long long* counts;
  int clear_input;
};
struct copy_args {
  const double* a;
  double* b;
  long n;
};
struct snap_args {
  const double* U;
  double* snapU;
  long KN;
  double g;
  const double* Bx;
  const double* By;
  const double* Bz;
  double* snapB;
  long G;
  int* flag;
};

// flag[0]: the attempt's reject word (bit 0: an inadmissible raw average), which the stage kernels
// test to skip the rest of a failed attempt; flag[1]: the entry check's word (bit 1: an inadmissible
// input), cleared at entry and copied into flag[0] at the start of every attempt so that an attempt
// on an inadmissible input does no work.
__global__ void k_reset_attempt(int* flag, unsigned long long* counts, int clear_input) {
  if (threadIdx.x == 0) {
    if (clear_input) flag[1] = 0;
    flag[0] = flag[1];
    counts[0] = 0; counts[1] = 0; counts[2] = 0;
  }
}

__global__ void k_copy(const double* __restrict__ a, double* __restrict__ b, long n) {
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) b[k] = a[k];
}

// ---------------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------------
#define DISPATCH_P(p, F) \
  switch (p) { case 1: F(1); break; case 2: F(2); break; case 3: F(3); break; \
               case 4: F(4); break; case 5: F(5); break; case 6: F(6); break; default: return -4; }

hipEvent_t* timing_slot(mhd25_ctx* c, int kid, int inner = 0);
static int eb_of(int p) { return 256 / ((p + 1) * (p + 1)); }
// Small meshes, by the elements of a launch (five for every compute unit).  The stage: at 32^2 elements the node form takes
// 7.1 (N = 3), 8.7, 10.0, 11.2 us (6) and the line form 7.9, 9.7, 12.2, 17.6; at 40^2 they are 8.1, 9.8, 12.1, 14.6
// against 8.0, 10.1, 11.7, 14.2, and beyond that the line form is ahead.  Below N = 3 it always is (5.5 us at 16^2, N = 1).
// A batch's launches cover a whole degree group, whose form goes by their sum: all forms give the same bits.
#ifndef MHD_SMALL_MESH
#define MHD_SMALL_MESH 1280L
#endif
static bool node_stage(const mhd25_ctx* c) { return c->p >= 3 && c->launch_elements <= MHD_SMALL_MESH; }
// The stage map in one launch.  N = 4 to 6: ahead up to about 56^2 (11.9, 15.0, 16.5 us at 48^2 against 13.7, 16.6, 22.2; 14.3,
// 18.1, 21.6 at 64^2 against 14.0, 17.6, 23).  N = 2 and 3: 9.2 and 11.4 us against 9.6 and 11.0 in two launches up to
// 32^2, 13.8 against 11.1 at 48^2 (N = 3).  On a mesh of one element's width a tile of the sensor is mostly outside
// the mesh: 65536 x 1, N = 4 77 against 79 + 30 us, N = 6 240 against 204 + 71 us.
static bool one_launch_map(const mhd25_ctx* c) {
  const long most = c->p >= 4 ? 5 * MHD_SMALL_MESH / 2 : c->p >= 2 ? MHD_SMALL_MESH : 0;
  return c->opt.oe_hydro && (c->launch_elements <= most || c->mp.nx == 1 || c->mp.ny == 1);
}
// threads per block of the hydro stage kernel: the tuned value if set, else 128.  256 take 906 against 885 us at 1024^2,
// N = 4 (the halves of a block wait for each other longer), at 128^2 1 to 4 % less for N = 1 and 3 to 6 and 9 to 18 % more at
// 24^2.
static int stage_block(const mhd25_ctx* c) { return c->hydro_bs == 256 ? 256 : 128; }
static long stage_blocks(const mhd25_ctx* c, int bs) {
  const long eb = node_stage(c) ? bs / (2 * c->nn) : bs / 2 / c->np;
  return (c->mp.K + eb - 1) / eb;
}
template <int P, int MODE>
static void launch_stage(mhd25_ctx* c, const double* Us, const double* Un, double* out, double* stats, int* flag, double ca,
                         double cb, double tau) {
  const int bs = stage_block(c);
  const dim3 grid(stage_blocks(c, bs));
#define GO(K) hipLaunchKernelGGL(K, grid, dim3(bs), 0, c->stream, Us, Un, out, stats, flag, c->d_ht, c->mp, ca, cb, tau, c->opt.iface_flux)
  if constexpr (P >= 3)
    if (node_stage(c)) {
      if (bs == 128) GO((k_hydro_stage_node<P, MODE, 128>));
      else GO((k_hydro_stage_node<P, MODE, 256>));
      return;
    }
  if (bs == 128) GO((k_hydro_stage<P, MODE, 128>));
  else GO((k_hydro_stage<P, MODE, 256>));
#undef GO
}

static int check(mhd25_ctx* c, hipError_t e, const char* what) {
  if (e != hipSuccess) { c->err = std::string(what) + ": " + hipGetErrorString(e); return -2; }
  return 0;
}

// row and column reductions of nc-component element records (nc = 1..5), then the global one
static int launch_reductions(mhd25_ctx* c, const double* stats, int nc, const int* flag) {
  const dim3 grid(c->mp.ny + (c->mp.nx + LRC - 1) / LRC);
  if (c->rec) {
    rt_record(c, RT_LINE_REDUCE, nc, grid.x,
              line_reduce_args{stats, c->lines, c->mp.nx, c->mp.ny, c->mp.bx, c->mp.by, flag});
    rt_record(c, RT_GLOBAL_REDUCE, nc, 1, global_reduce_args{c->lines, c->glob, c->mp.by, flag});
    return 0;
  }
#define LR(NC)                                                                                                    \
  hipLaunchKernelGGL((k_line_reduce<NC>), grid, dim3(256), 0, c->stream, stats, c->lines, c->mp.nx, c->mp.ny,    \
                     c->mp.bx, c->mp.by, flag);                                                                   \
  hipLaunchKernelGGL((k_global_reduce<NC>), dim3(1), dim3(256), 0, c->stream, c->lines, c->glob, c->mp.by, flag)
  switch (nc) { case 1: LR(1); break; case 2: LR(2); break; case 3: LR(3); break; case 4: LR(4); break;
                case 5: LR(5); break; default: c->err = "line reduction: unsupported component count"; return -2; }
#undef LR
  return 0;
}

int hydro_rhs(mhd25_ctx* c, const double* U, double* dU) {
#define L0(P) launch_stage<P, 0>(c, U, U, dU, nullptr, nullptr, 0.0, 1.0, 0.0)
  DISPATCH_P(c->p, L0);
#undef L0
  return check(c, hipGetLastError(), "rhs_hydro launch");
}

// raw stage + statistics + line/global reductions (the OE sensor's only: without OE nothing reads them, and on a
// 16^2 mesh they were a quarter of a step)
int hydro_stage_a(mhd25_ctx* c, const double* Us, const double* Un, double* Ust, double ca, double cb, double tau) {
  if (c->rec) {
    const int bs = stage_block(c);
    rt_record(c, RT_HYDRO_STAGE, (node_stage(c) ? 10000 : 0) + c->p * 1000 + bs, stage_blocks(c, bs),
              hydro_stage_args{Us, Un, Ust, c->stats, c->d_flag, c->d_ht, c->mp, ca, cb, tau, c->opt.iface_flux});
    return c->opt.oe_hydro ? launch_reductions(c, c->stats, 5, c->d_flag) : 0;
  }
  hipEvent_t* ev = c->timing ? timing_slot(c, 0) : nullptr;
  if (ev) hipEventRecord(ev[0], c->stream);
#define L1(P) launch_stage<P, 1>(c, Us, Un, Ust, c->stats, c->d_flag, ca, cb, tau)
  DISPATCH_P(c->p, L1);
#undef L1
  if (ev) hipEventRecord(ev[1], c->stream);
  int r = check(c, hipGetLastError(), "hydro stage launch");
  if (r) return r;
  if (!c->opt.oe_hydro) return 0;
  if (const int rl = launch_reductions(c, c->stats, 5, c->d_flag)) return rl;
  return check(c, hipGetLastError(), "reduce launch");
}

int line_global_reduce(mhd25_ctx* c, const double* stats, int nc, const int* flag) {
  if (const int r = launch_reductions(c, stats, nc, flag)) return r;
  return check(c, hipGetLastError(), "reduce launch");
}

int hydro_stats_only(mhd25_ctx* c, const double* U, int* flag) {
  const long blocks = (c->mp.K + eb_of(c->p) - 1) / eb_of(c->p);
#define LS(P) hipLaunchKernelGGL((k_elem_stats<P>), dim3(blocks), dim3(256), 0, c->stream, U, c->stats, flag, c->d_ht, c->mp)
  DISPATCH_P(c->p, LS);
#undef LS
  if (const int rl = launch_reductions(c, c->stats, 5, nullptr)) return rl;
  return check(c, hipGetLastError(), "stats launch");
}

// The stage map: the OE sensor (damping factors, into the context's dfac), then the map itself.
// rho_o, e_o, u_o: optional primitive outputs (all null or all set)
int hydro_stage_b(mhd25_ctx* c, const double* Ust, double* Uout, double tau, const int* flag, double* rho_o,
                  double* e_o, double* u_o) {
  const long sblocks = (long)((c->mp.nx + HS<1>::TX - 1) / HS<1>::TX) * ((c->mp.ny + HS<1>::TY - 1) / HS<1>::TY);
  const long blocks = (c->mp.K + OM<1>::EB - 1) / OM<1>::EB;
  const long lblocks = (c->mp.K + ML_BS / c->nn - 1) / (ML_BS / c->nn);
  const bool one = one_launch_map(c);
  if (c->rec && one) {  // (a plan's runs share one sequence of launches: the sensor's place is kept, with no block)
    rt_record(c, RT_HYDRO_SENSOR, 0, 0, hydro_sensor_args{});
    rt_record(c, RT_OE_PP, 10 + c->p, lblocks,
              hydro_map_lines_args{Ust, Uout, c->stats, c->lines, c->glob, c->d_flags, c->d_counts, flag, c->d_ht, c->mp,
                                   tau, c->opt.s_H, c->opt.pp, rho_o, e_o, u_o});
    return 0;
  }
  if (c->rec) {
    if (c->opt.oe_hydro)
      rt_record(c, RT_HYDRO_SENSOR, c->p, sblocks,
                hydro_sensor_args{Ust, c->stats, c->lines, c->glob, c->dfac, flag, c->d_ht, c->mp, tau, c->opt.s_H});
    rt_record(c, RT_OE_PP, c->p, blocks,
              hydro_oe_pp_args{Ust, Uout, c->stats, c->dfac, c->d_flags, c->d_counts, flag, c->d_ht, c->mp,
                               c->opt.oe_hydro, c->opt.pp, rho_o, e_o, u_o});
    return 0;
  }
  hipEvent_t* ev = c->timing ? timing_slot(c, 1, 1) : nullptr;
  if (ev) hipEventRecord(ev[0], c->stream);
  if (one) {
#define LM(P) hipLaunchKernelGGL((k_hydro_map_lines<P>), dim3(lblocks), dim3(ML_BS), 0, c->stream, Ust, Uout, c->stats, \
                                 c->lines, c->glob, c->d_flags, c->d_counts, flag, c->d_ht, c->mp, tau, c->opt.s_H, \
                                 c->opt.pp, rho_o, e_o, u_o)
    DISPATCH_P(c->p, LM);
#undef LM
    if (ev) hipEventRecord(ev[1], c->stream);
    return check(c, hipGetLastError(), "stage map launch");
  }
  if (c->opt.oe_hydro) {
    hipEvent_t* sev = c->timing ? timing_slot(c, 8) : nullptr;
    if (sev) hipEventRecord(sev[0], c->stream);
#define LS(P) hipLaunchKernelGGL((k_hydro_sensor<P>), dim3(sblocks), dim3(HS<P>::BS), 0, c->stream, Ust, c->stats, c->lines, \
                                 c->glob, c->dfac, flag, c->d_ht, c->mp, tau, c->opt.s_H)
    DISPATCH_P(c->p, LS);
#undef LS
    if (sev) hipEventRecord(sev[1], c->stream);
  }
#define LB(P) hipLaunchKernelGGL((k_hydro_oe_pp<P>), dim3(blocks), dim3(OM<P>::BS), 0, c->stream, Ust, Uout, c->stats, \
                                 c->dfac, c->d_flags, c->d_counts, flag, c->d_ht, c->mp, c->opt.oe_hydro, c->opt.pp, rho_o, \
                                 e_o, u_o)
  DISPATCH_P(c->p, LB);
#undef LB
  if (ev) hipEventRecord(ev[1], c->stream);
  return check(c, hipGetLastError(), "stage map launch");
}

int reset_attempt(mhd25_ctx* c) {
  if (c->rec) { rt_record(c, RT_RESET, 0, 1, reset_args{c->d_flag, c->d_counts, 0}); return 0; }
  hipLaunchKernelGGL(k_reset_attempt, dim3(1), dim3(64), 0, c->stream, c->d_flag, c->d_counts, 0);
  return check(c, hipGetLastError(), "reset launch");
}

static long flat_blocks(long n) {
  long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  return blocks < 1 ? 1 : blocks;
}

// clears the entry word flag[1] (and the attempt's word and counters)
int entry_clear(mhd25_ctx* c) {
  hipLaunchKernelGGL(k_reset_attempt, dim3(1), dim3(64), 0, c->stream, c->d_flag, c->d_counts, 1);
  return check(c, hipGetLastError(), "entry clear launch");
}

// entry snapshot of U (and of the magnetic grids when B is set) into snapU / saveB with the
// admissibility test; clears and then sets the entry word flag[1]
int entry_snapshot(mhd25_ctx* c, const double* U, double* snapU, const double* const* B, double* saveB) {
  const long KN = c->mp.K * c->nn, G = B ? c->G : 0;
  const double *Bx = B ? B[0] : nullptr, *By = B ? B[1] : nullptr, *Bz = B ? B[2] : nullptr;
  if (c->rec) {
    rt_record(c, RT_RESET, 0, 1, reset_args{c->d_flag, c->d_counts, 1});
    rt_record(c, RT_SNAP, 0, flat_blocks(KN), snap_args{U, snapU, KN, c->mp.gamma, Bx, By, Bz, saveB, G, c->d_flag});
    return 0;
  }
  hipLaunchKernelGGL(k_reset_attempt, dim3(1), dim3(64), 0, c->stream, c->d_flag, c->d_counts, 1);
  hipLaunchKernelGGL(k_snap_check, dim3(flat_blocks(KN)), dim3(256), 0, c->stream, U, snapU, KN, c->mp.gamma, Bx, By, Bz,
                     saveB, G, c->d_flag);
  return check(c, hipGetLastError(), "entry snapshot launch");
}

int hydro_face_map(mhd25_ctx* c, int32_t* nbr, int32_t* fmap) {
  const long blocks = (4 * c->mp.K + 255) / 256;
#define FM(P) hipLaunchKernelGGL((k_face_map<P>), dim3(blocks), dim3(256), 0, c->stream, nbr, fmap, c->mp)
  DISPATCH_P(c->p, FM);
#undef FM
  return check(c, hipGetLastError(), "face map launch");
}

int dcopy(mhd25_ctx* c, const double* a, double* b, long n) {
  long blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  if (c->rec) { rt_record(c, RT_COPY, 0, blocks, copy_args{a, b, n}); return 0; }
  hipLaunchKernelGGL(k_copy, dim3(blocks), dim3(256), 0, c->stream, a, b, n);
  return check(c, hipGetLastError(), "copy launch");
}

// ---------------------------------------------------------------------------------------------
// Run-table kernels of the small and flat kernels (argument structs per run) and the dispatcher of
// this file's run-table launches.
// ---------------------------------------------------------------------------------------------
__global__ void k_reset_rt(const reset_args* __restrict__ A, int nr) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nr) return;
  const reset_args& a = A[r];
  if (a.clear_input) gl(a.flag)[1] = 0;
  gl(a.flag)[0] = gl(a.flag)[1];
  gl(a.counts)[0] = 0; gl(a.counts)[1] = 0; gl(a.counts)[2] = 0;
}

// flat kernels: run r owns blocks boff[r] .. boff[r+1) and strides over its n entries with them
__global__ __launch_bounds__(256) void k_copy_rt(const copy_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const copy_args& a = A[r];
  const long stride = (long)(boff[r + 1] - boff[r]) * blockDim.x;
  for (long k = (long)(blockIdx.x - boff[r]) * blockDim.x + threadIdx.x; k < a.n; k += stride) gl(a.b)[k] = gl(a.a)[k];
}

__global__ __launch_bounds__(256) void k_snap_check_rt(const snap_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const snap_args& a = A[r];
  const long k0 = (long)(blockIdx.x - boff[r]) * blockDim.x + threadIdx.x, dk = (long)(boff[r + 1] - boff[r]) * blockDim.x;
  for (long n = k0; n < a.KN; n += dk) snap_check_node(gl(a.U), gl(a.snapU), a.KN, a.g, gl(a.flag), n);
  for (long k = k0; k < a.G; k += dk) snap_check_B(gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.snapB), a.G, gl(a.flag), k);
}

template <int P>
static void launch_stage_rt(bool node, int bs, dim3 g, hipStream_t s, const hydro_stage_args* A, const int* dboff, int nr) {
  if constexpr (P >= 3)
    if (node) {
      if (bs == 128) hipLaunchKernelGGL((k_hydro_stage_node_rt<P, 1, 128>), g, dim3(128), 0, s, A, dboff, nr);
      else hipLaunchKernelGGL((k_hydro_stage_node_rt<P, 1, 256>), g, dim3(256), 0, s, A, dboff, nr);
      return;
    }
  if (bs == 128) hipLaunchKernelGGL((k_hydro_stage_rt<P, 1, 128>), g, dim3(128), 0, s, A, dboff, nr);
  else hipLaunchKernelGGL((k_hydro_stage_rt<P, 1, 256>), g, dim3(256), 0, s, A, dboff, nr);
}

int hydro_rt_launch(const RtRecord& h, const void* dargs, const int* dboff, int nr, long nblocks, hipStream_t s) {
  const dim3 g((unsigned)nblocks);
  switch (h.kind) {
    case RT_HYDRO_STAGE: {
      const int P = h.key / 1000 % 10, bs = h.key % 1000;
      const bool node = h.key >= 10000;
      const hydro_stage_args* A = (const hydro_stage_args*)dargs;
#define RS(P_) launch_stage_rt<P_>(node, bs, g, s, A, dboff, nr)
      DISPATCH_P(P, RS);
#undef RS
      break;
    }
    case RT_HYDRO_SENSOR: {
      const hydro_sensor_args* A = (const hydro_sensor_args*)dargs;
#define RV(P_) hipLaunchKernelGGL((k_hydro_sensor_rt<P_>), g, dim3(HS<P_>::BS), 0, s, A, dboff, nr)
      DISPATCH_P(h.key, RV);
#undef RV
      break;
    }
    case RT_OE_PP: {
      if (h.key > 10) {
        const hydro_map_lines_args* A = (const hydro_map_lines_args*)dargs;
#define RM(P_) hipLaunchKernelGGL((k_hydro_map_lines_rt<P_>), g, dim3(ML_BS), 0, s, A, dboff, nr)
        DISPATCH_P(h.key - 10, RM);
#undef RM
        break;
      }
      const hydro_oe_pp_args* A = (const hydro_oe_pp_args*)dargs;
#define RO(P_) hipLaunchKernelGGL((k_hydro_oe_pp_rt<P_>), g, dim3(OM<P_>::BS), 0, s, A, dboff, nr)
      DISPATCH_P(h.key, RO);
#undef RO
      break;
    }
    case RT_LINE_REDUCE: {
      const line_reduce_args* A = (const line_reduce_args*)dargs;
#define RL(NC) hipLaunchKernelGGL((k_line_reduce_rt<NC>), g, dim3(256), 0, s, A, dboff, nr)
      switch (h.key) { case 1: RL(1); break; case 2: RL(2); break; case 3: RL(3); break; case 4: RL(4); break;
                       case 5: RL(5); break; default: return -2; }
#undef RL
      break;
    }
    case RT_GLOBAL_REDUCE: {
      const global_reduce_args* A = (const global_reduce_args*)dargs;
#define RG(NC) hipLaunchKernelGGL((k_global_reduce_rt<NC>), g, dim3(256), 0, s, A, dboff, nr)
      switch (h.key) { case 1: RG(1); break; case 2: RG(2); break; case 3: RG(3); break; case 4: RG(4); break;
                       case 5: RG(5); break; default: return -2; }
#undef RG
      break;
    }
    case RT_RESET:
      hipLaunchKernelGGL(k_reset_rt, dim3((nr + 63) / 64), dim3(64), 0, s, (const reset_args*)dargs, nr);
      break;
    case RT_COPY:
      hipLaunchKernelGGL(k_copy_rt, g, dim3(256), 0, s, (const copy_args*)dargs, dboff, nr);
      break;
    case RT_SNAP:
      hipLaunchKernelGGL(k_snap_check_rt, g, dim3(256), 0, s, (const snap_args*)dargs, dboff, nr);
      break;
    default:
      return 1;  // not a kind of this file
  }
  return hipGetLastError() == hipSuccess ? 0 : -2;
}
