// Magnetic-velocity subflow kernels for gfx950 (section "Magnetic--velocity subflow:
// compatible finite elements").
//
// Element-local kernels use one block per tile of EB elements; element data are staged in LDS.  Shared
// degrees of freedom are assembled by the tile that owns them, in a fixed order (no floating-point
// atomics), with the lumped weights of eq. quad-hcurl-element and eq. quad-cg-element.
#include <cfloat>
#include <mutex>
#include <string>

#include "common.h"
#include "xcd.h"
#include "jumps.h"
#include "rsqrt.h"

namespace {

constexpr double EPSM = 2.220446049250313e-16;

template <int P, int M, int BS = 256>
struct MC {
  static constexpr int NP = P + 1, NN = NP * NP, A = M + 2, B = M + 1, AA = A * A, AB = A * B, BB = B * B;
  static constexpr int NT = NN > AA ? NN : AA;
  static constexpr int EB = BS / NT;
};

__device__ __forceinline__ long wrapl(long a, long n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// global index of local node (i, j) of element (ex, ey) on a magnetic grid (32-bit arithmetic: a
// grid holds fewer than 2^29 nodes, which mhd25_init guarantees)
__device__ __forceinline__ long gix(const MeshP& mp, int B, long ex, long ey, int i, int j) {
  const int NX = mp.nx * B, NY = mp.ny * B;
  int gx = (int)ex * B + i, gy = (int)ey * B + j;
  if (gx >= NX) gx -= NX;
  if (gy >= NY) gy -= NY;
  return (long)(gy * NX + gx);
}

// ---------------------------------------------------------------------------------------------
// Reconstruction of J (eq. mag-current-proj) and E (eq. mag-electric-proj) on the auxiliary grids.
//
// Both are assembled on tiles of TX x TY elements: a task forms one grid row of an element (row tasks of
// the W rows, for the x and z components, on the block's first waves; of the Gauss rows, for the y
// component, on the others).  At the shared node of a row it adds the left element's contribution, whose
// operands it reads too; row A-1 of the element below a tile element is a task of the tile, added to that
// element's row 0 through LDS.  So every node is written once, by its owner, and no per-element loads pass
// through memory: with a load kernel and a gather per field these moved 1 040 B more per element and
// field at k = 3.  The 1D operators along x are scalars (compile-time indices), those along y are the
// task's own row of the table.
//
// Lumped weights: with W_i the assembled 1D weight of node i, the tables RWQ.. hold the 1D operators with
// row i divided by W_i (|J_K| cancels).
// ---------------------------------------------------------------------------------------------
// S: tile shape, 0 TX x TY; on meshes of one element's width, where such a tile is mostly outside the mesh, the same
// number of elements in a row (1) or a column (2).  On 65536 x 1 elements with resistivity k_J takes 37 and k_E 79 us
// (N = k = 4) where the 5 x 4 tiles took 68 and 221, at N = k = 6 88 and 230 against 167 and 702.
template <int M, bool R2, int S>
struct RT {
  static constexpr int A = M + 2, B = M + 1;
  // tile sizes that fill the row tasks' waves: A TE of the W rows, B TE of the Gauss rows
  static constexpr int SX = M == 2 || M >= 5 ? 4 : 5, SY = M == 3 ? 5 : 4, TE = SX * SY;
  static constexpr int TX = S == 0 ? SX : (S == 1 ? TE : 1), TY = S == 0 ? SY : (S == 1 ? 1 : TE);
  static constexpr int WW = (A * TE + 63) / 64 * 64;  // threads of the W rows (whole waves)
  static constexpr int BS = R2 ? WW : WW + (B * TE + 63) / 64 * 64;
};

// A patch of NR x NC nodes of a periodic magnetic grid on its way to LDS: the loads of several patches
// are issued before the first is waited for.  In LDS node (row y B + j, column x B + i) lies at
// y RS + j PITCH + i W + x with RS = TX (mod 16), so that 16 lanes of neighbouring elements, TX to a row, read
// 16 neighbouring doubles, all banks (in the grid's own order their stride of B doubles conflicts).
template <int NR, int NC, int B, int TX, int BS>
struct Patch {
  static constexpr int N = NR * NC, R = (N + BS - 1) / BS, W = (NC + B - 1) / B, PITCH = W * B;
  static constexpr int RS = B * PITCH + (TX - B * PITCH % 16 + 16) % 16, SIZE = (NR + B - 1) / B * RS;
  // offset of node (i, j) from its element's (x, y) (i = B or j = B: the next element's first node)
  static __device__ __forceinline__ constexpr int at(int i, int j = 0) { return (i < B ? i * W : 1) + (j < B ? j * PITCH : RS); }
  double v[R];
  // nodes (gy0 + r, gx0 + c), r < nr, c < nc (at most one period away from the grid)
  __device__ __forceinline__ void load(const double* __restrict__ f, const MeshP& mp, int gx0, int gy0, int nc, int nr) {
    const int NXg = mp.nx * B, NYg = mp.ny * B;
    const auto rs = node_rsrc(f, (long)NXg * NYg);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int n = threadIdx.x + k * BS, r = n / NC, c = n - r * NC;
      v[k] = 0.0;
      if (r < nr && c < nc) v[k] = bld(rs, (unsigned)(wrap32(gy0 + r, NYg) * NXg + wrap32(gx0 + c, NXg)) * 8u);
    }
  }
  __device__ __forceinline__ void store(double* s) const {
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int n = threadIdx.x + k * BS, r = n / NC, c = n - r * NC;
      if (n < N) s[r / B * RS + r % B * PITCH + c % B * W + c / B] = v[k];
    }
  }
};

// sum_k t[k] f[k * step] of an N-term row
template <int N>
__device__ __forceinline__ double dot_col(const double* t, const double* f, int step) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < N; ++k) s = fma(t[k], f[k * step], s);
  return s;
}

// the same down N nodes of column i of an element at f in a patch
template <class Q, int N>
__device__ __forceinline__ double dot_patch(const double* t, const double* f, int i) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < N; ++k) s = fma(t[k], f[Q::at(i, k)], s);
  return s;
}

// The thread's row task: W row j (or Gauss row j) of tile element (lx, ly); ye is the element row it reads,
// ly, or ly - 1 for the row A-1 of the element below.
template <int M, bool R2, int S>
struct RowTask {
  bool w, act, below;
  int j, lx, ly, ye, el;
  __device__ __forceinline__ RowTask(int tw, int th) {
    using C = RT<M, R2, S>;
    w = R2 || __builtin_amdgcn_readfirstlane(threadIdx.x < C::WW ? 1 : 0);
    const int t = threadIdx.x - (w ? 0 : C::WW);
    j = t / C::TE; el = t - j * C::TE;
    ly = el / C::TX; lx = el - ly * C::TX;
    act = j < (w ? C::A : C::B) && lx < tw && ly < th;
    below = w && j == C::A - 1;
    ye = below ? ly - 1 : ly;
  }
};

// J: int B_x d_y phi - B_y d_x phi with the (m+2)-point Gauss rule (z), int B_z (-d_y psi) and int B_z d_x psi
// with the (m+1)-point rule (x, y), each as one operator per direction.
// The mass matrix's rows are summed from the diagonal on.  The order is one of rounding, but J of a uniform field is
// rounding alone, and so is ||div B|| at the end of the rotor run, which its test holds to the published 4.60e-12 within
// 5 %: this order gives 0.96 and 0.97 of it (without and with A.R.), the plain one 0.94, the reversed 1.33, even then
// odd terms 1.43.
// Measured: 1024^2, N = 4, k = 3: 0.66 (load kernel and gather) -> 0.29 ms; 128^2, N = k = 4: 28 -> 13 us.  Bound by the
// latency of its staging loads and barriers (0.84 GB moved).
template <int M, bool R2, int S>
__device__ __forceinline__ void J_body(const double* __restrict__ Bx, const double* __restrict__ By,
                                       const double* __restrict__ Bz, double* __restrict__ Jx, double* __restrict__ Jy,
                                       double* __restrict__ Jz, const MagTab* __restrict__ T, const MeshP& mp, int blk) {
  using C = RT<M, R2, S>;
  constexpr int A = C::A, B = C::B, TX = C::TX, TY = C::TY, TE = C::TE, BS = C::BS;
  // the tile's elements, the column left of it and the row below
  using PX = Patch<(TY + 1) * B, (TX + 1) * B + 1, B, TX, BS>;
  using PY = Patch<(TY + 1) * B + 1, (TX + 1) * B, B, TX, BS>;
  using PZ = Patch<(TY + 1) * B, (TX + 1) * B, B, TX, BS>;
  __shared__ double sx[PX::SIZE], sy[PY::SIZE], sz[R2 ? 1 : PZ::SIZE], sbel[2][TE][B];
  int tx0, ty0;
  tile_of(blk, (mp.nx + TX - 1) / TX, (mp.ny + TY - 1) / TY, tx0, ty0);
  tx0 *= TX; ty0 *= TY;
  const int tw = mp.nx - tx0 < TX ? mp.nx - tx0 : TX, th = mp.ny - ty0 < TY ? mp.ny - ty0 : TY;
  {
    PX px;
    PY py;
    const int gx0 = (tx0 - 1) * B, gy0 = (ty0 - 1) * B;
    px.load(Bx, mp, gx0, gy0, (tw + 1) * B + 1, (th + 1) * B);
    py.load(By, mp, gx0, gy0, (tw + 1) * B, (th + 1) * B + 1);
    if constexpr (!R2) {
      PZ pz;
      pz.load(Bz, mp, gx0, gy0, (tw + 1) * B, (th + 1) * B);
      pz.store(sz);
    }
    px.store(sx);
    py.store(sy);
  }
  const RowTask<M, R2, S> k(tw, th);
  const int gx = (tx0 + k.lx) * B, gy = (ty0 + k.ly) * B + k.j, NXg = mp.nx * B;
  double tq[A], td[B], tv[B];  // rows j of the tables along y
  if (k.act) {
#pragma unroll
    for (int i = 0; i < A; ++i) tq[i] = k.w ? T->RWQ[k.j][i] : 0.0;
#pragma unroll
    for (int i = 0; i < B; ++i) { td[i] = k.w ? T->RDG[k.j][i] : 0.0; tv[i] = k.w ? T->RDV[k.j][i] : T->I_V_G[k.j][i]; }
  }
  __syncthreads();
  // the task's element in the patches
  const double* const xe = sx + (k.ye + 1) * PX::RS + k.lx + 1;
  const double* const yq = sy + (k.ye + 1) * PY::RS + k.lx + 1;
  const double* const ze = sz + (k.ye + 1) * PZ::RS + k.lx + 1;
  const double sX = 2.0 * mp.rhx, sY = 2.0 * mp.rhy;
  double z[B], x[B];
  if (k.act && k.w) {
    double c[A], cl[B];  // Bx summed along y; cl: the left element's (its last node is this one's first)
#pragma unroll
    for (int i = 0; i < A; ++i) c[i] = dot_patch<PX, B>(td, xe, i);
#pragma unroll
    for (int i = 0; i < B; ++i) cl[i] = dot_patch<PX, B>(td, xe - 1, i);
    double d[B], dl[B];  // By
#pragma unroll
    for (int i = 0; i < B; ++i) {
      d[i] = dot_patch<PY, A>(tq, yq, i);
      dl[i] = dot_patch<PY, A>(tq, yq - 1, i);
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      double s = 0.0, t = 0.0;
#pragma unroll
      for (int q = 0; q < A; ++q) s = fma(T->RWQ[i][(i + q) % A], c[(i + q) % A], s);
#pragma unroll
      for (int q = 0; q < B; ++q) t = fma(T->RDG[i][q], d[q], t);
      if (i == 0) {
        s = fma(T->RWQ[A - 1][A - 1], c[0], s);
#pragma unroll
        for (int q = 0; q < B; ++q) {
          s = fma(T->RWQ[A - 1][q], cl[q], s);
          t = fma(T->RDG[A - 1][q], dl[q], t);
        }
      }
      z[i] = sY * s - sX * t;
    }
    if constexpr (!R2) {
      double f[B];
#pragma unroll
      for (int i = 0; i < B; ++i) f[i] = dot_patch<PZ, B>(tv, ze, i);
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < B; ++q) s = fma(T->I_V_G[i][q], f[q], s);
        x[i] = -sY * s;
      }
    }
    if (k.below)
#pragma unroll
      for (int i = 0; i < B; ++i) { sbel[0][k.el][i] = z[i]; sbel[1][k.el][i] = R2 ? 0.0 : x[i]; }
  }
  if constexpr (!R2) {
    if (k.act && !k.w) {
      double f[B], fl[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        f[i] = dot_patch<PZ, B>(tv, ze, i);
        fl[i] = dot_patch<PZ, B>(tv, ze - 1, i);
      }
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < B; ++q) s = fma(T->RDV[i][q], f[q], s);
        if (i == 0)
#pragma unroll
          for (int q = 0; q < B; ++q) s = fma(T->RDV[A - 1][q], fl[q], s);
        Jy[(long)gy * NXg + gx + i] = sX * s;
      }
    }
  }
  __syncthreads();
  if (k.act && k.w && !k.below) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const long g = (long)gy * NXg + gx + i;
      Jz[g] = k.j == 0 ? z[i] + sbel[0][k.el][i] : z[i];
      if (!R2) Jx[g] = k.j == 0 ? x[i] + sbel[1][k.el][i] : x[i];
    }
  }
}

// e + eta j; an element without resistivity is not touched by its J, also where that is infinite or NaN
__device__ __forceinline__ double add_eta(double eta, double j, double e) { return eta != 0.0 ? fma(eta, j, e) : e; }

// E: -u x B at the nodes, averaged over the elements that share the node (their lumped weights are equal),
// plus eta_K sum_q M_q J(x_q) . phi_a(x_q) by the degree-p GLL rule, i.e. the 1D operators RWP / RGP applied
// to J; blocks whose elements all have eta = 0 skip that term.
// Measured: 1024^2, N = 4, k = 3, with resistivity: 1.08 (load kernel and gather) -> 0.55 ms; 128^2, N = k = 4, without:
// 36 -> 17.5 us.  Bound by LDS reads and latency (1.5 GB moved where few elements are
// resistive).
template <int P, int M, bool R2, int S>
__device__ __forceinline__ void E_body(const double* __restrict__ u, const double* __restrict__ Bx,
                                       const double* __restrict__ By, const double* __restrict__ Bz,
                                       const double* __restrict__ Jx, const double* __restrict__ Jy,
                                       const double* __restrict__ Jz, const double* __restrict__ eta,
                                       double* __restrict__ Ex, double* __restrict__ Ey, double* __restrict__ Ez,
                                       const MagTab* __restrict__ T, const MeshP& mp, int blk) {
  using C = RT<M, R2, S>;
  constexpr int A = C::A, B = C::B, TX = C::TX, TY = C::TY, TE = C::TE, BS = C::BS;
  constexpr int NP = P + 1, NN = NP * NP, ES = NN | 1, NU = R2 ? 2 : 3;
  constexpr int NE = (TX + 1) * (TY + 1);  // staged elements: the tile's, the column left of it, the row below
  using PX = Patch<(TY + 1) * B, TX * B, B, TX, BS>;  // B_x: the row below
  using PY = Patch<TY * B, (TX + 1) * B, B, TX, BS>;  // B_y: the column left
  using PZ = Patch<(TY + 1) * B, (TX + 1) * B, B, TX, BS>;
  using QX = Patch<(TY + 1) * B + 1, TX * B, B, TX, BS>;  // J_x, J_y, J_z: the shared nodes of the last elements too
  using QY = Patch<TY * B, (TX + 1) * B + 1, B, TX, BS>;
  using QZ = Patch<(TY + 1) * B + 1, (TX + 1) * B + 1, B, TX, BS>;
  __shared__ double su[NU * NE * ES], sx[PX::SIZE], sy[PY::SIZE], sz[R2 ? 1 : PZ::SIZE], sbel[2][TE][B];
  __shared__ double jx[R2 ? 1 : QX::SIZE], jy[R2 ? 1 : QY::SIZE], jz[QZ::SIZE];
  int tx0, ty0;
  tile_of(blk, (mp.nx + TX - 1) / TX, (mp.ny + TY - 1) / TY, tx0, ty0);
  tx0 *= TX; ty0 *= TY;
  const int tw = mp.nx - tx0 < TX ? mp.nx - tx0 : TX, th = mp.ny - ty0 < TY ? mp.ny - ty0 : TY;
  const long KN = mp.K * NN;
  const int bx0 = tx0 * B, by0 = ty0 * B;
  const RowTask<M, R2, S> k(tw, th);
  // resistivity of the task's element and of the one left of it
  double et = 0.0, etl = 0.0;
  if (eta && k.act) {
    const int row = wrap32(ty0 + k.ye, mp.ny) * mp.nx;
    et = eta[row + tx0 + k.lx];
    etl = eta[row + wrap32(tx0 + k.lx - 1, mp.nx)];
  }
  {
    constexpr int NR = (NE * NN + BS - 1) / BS;
    double v[NR][NU];
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = threadIdx.x + m * BS, s = n / NN, q = n - s * NN, y = s / (TX + 1), x = s - y * (TX + 1);
      if (s < NE && x <= tw && y <= th) {
        const unsigned o = ((unsigned)(wrap32(ty0 + y - 1, mp.ny) * mp.nx + wrap32(tx0 + x - 1, mp.nx)) * NN + q) * 8u;
#pragma unroll
        for (int d = 0; d < NU; ++d) v[m][d] = bld(node_rsrc(u + d * KN, KN), o);
      }
    }
    PX px;
    PY py;
    px.load(Bx, mp, bx0, by0 - B, tw * B, (th + 1) * B);
    py.load(By, mp, bx0 - B, by0, (tw + 1) * B, th * B);
    if constexpr (!R2) {
      PZ pz;
      pz.load(Bz, mp, bx0 - B, by0 - B, (tw + 1) * B, (th + 1) * B);
      pz.store(sz);
    }
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = threadIdx.x + m * BS, s = n / NN, q = n - s * NN;
      if (s < NE)
#pragma unroll
        for (int d = 0; d < NU; ++d) su[(d * NE + s) * ES + q] = v[m][d];
    }
    px.store(sx);
    py.store(sy);
  }
  bool res = false;
  if (eta) {
    res = __syncthreads_or(et != 0.0 || etl != 0.0);
    if (res) {
      QZ pz;
      pz.load(Jz, mp, bx0 - B, by0 - B, (tw + 1) * B + 1, (th + 1) * B + 1);
      if constexpr (!R2) {
        QX px;
        QY py;
        px.load(Jx, mp, bx0, by0 - B, tw * B, (th + 1) * B + 1);
        py.load(Jy, mp, bx0 - B, by0, (tw + 1) * B + 1, th * B);
        px.store(jx);
        py.store(jy);
      }
      pz.store(jz);
    }
  }
  double tp[NP], tg[B], tv[B];  // rows j of the interpolations along y: of u, of B_x (W rows), of B_z
  if (k.act) {
#pragma unroll
    for (int q = 0; q < NP; ++q) tp[q] = k.w ? T->I_P_W[k.j][q] : T->I_P_G[k.j][q];
#pragma unroll
    for (int q = 0; q < B; ++q) { tg[q] = k.w ? T->I_G_W[k.j][q] : 0.0; tv[q] = k.w ? T->I_V_W[k.j][q] : T->I_V_G[k.j][q]; }
  }
  __syncthreads();
  const int gx = (tx0 + k.lx) * B, gy = (ty0 + k.ly) * B + k.j, NXg = mp.nx * B;
  // the task's element and the one left of it in su (row 0 of the staged elements is the row below the tile)
  const double* ue = su + ((k.ye + 1) * (TX + 1) + k.lx + 1) * ES;
  const double* ul = ue - ES;
  const double* const ze = sz + (k.ye + 1) * PZ::RS + k.lx + 1;  // B_z of the element
  double z[B], x[B];
  if (k.act && k.w) {
    const double cj = k.j == 0 || k.j == A - 1 ? 0.5 : 1.0;
    double u0[NP], u1[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      u0[q] = dot_col<NP>(tp, ue + q, NP);
      u1[q] = dot_col<NP>(tp, ue + NE * ES + q, NP);
    }
    const double l0 = dot_col<NP>(tp, ul + P, NP), l1 = dot_col<NP>(tp, ul + NE * ES + P, NP);  // left, at x = +1
    double b1[B], bl = 0.0;  // B_y of the row at the Gauss nodes; the left element's at x = +1
    const double* yr = sy + k.ly * PY::RS + (k.below ? 0 : k.j) * PY::PITCH + k.lx + 1;
#pragma unroll
    for (int q = 0; q < B; ++q) {
      b1[q] = yr[PY::at(q)];
      bl = fma(T->I_G_W[A - 1][q], yr[PY::at(q) - 1], bl);
    }
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const double bx = dot_patch<PX, B>(tg, sx + (k.ye + 1) * PX::RS + k.lx, i);
      double ux = 0.0, uy = 0.0, by = 0.0;
#pragma unroll
      for (int q = 0; q < NP; ++q) { ux = fma(T->I_P_W[i][q], u0[q], ux); uy = fma(T->I_P_W[i][q], u1[q], uy); }
#pragma unroll
      for (int q = 0; q < B; ++q) by = fma(T->I_G_W[i][q], b1[q], by);
      z[i] = -(ux * by - uy * bx);
      if (i == 0) z[i] = 0.5 * (z[i] - (l0 * bl - l1 * bx));
      z[i] *= cj;
    }
    if constexpr (!R2) {
      double u2[NP], bz[B];
#pragma unroll
      for (int q = 0; q < NP; ++q) u2[q] = dot_col<NP>(tp, ue + 2 * NE * ES + q, NP);
#pragma unroll
      for (int q = 0; q < B; ++q) bz[q] = dot_patch<PZ, B>(tv, ze, q);
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double uy = 0.0, uz = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < NP; ++q) { uy = fma(T->I_P_G[i][q], u1[q], uy); uz = fma(T->I_P_G[i][q], u2[q], uz); }
#pragma unroll
        for (int q = 0; q < B; ++q) b = fma(T->I_V_G[i][q], bz[q], b);
        x[i] = -cj * (uy * b - uz * b1[i]);
      }
    }
    if (res) {
      double tw_[A];
#pragma unroll
      for (int q = 0; q < A; ++q) tw_[q] = T->RWP[k.j][q];
      const double* r = jz + (k.ye + 1) * QZ::RS + k.lx + 1;
      double c[A], cl[B];
#pragma unroll
      for (int q = 0; q < A; ++q) c[q] = dot_patch<QZ, A>(tw_, r, q);
#pragma unroll
      for (int q = 0; q < B; ++q) cl[q] = dot_patch<QZ, A>(tw_, r - 1, q);
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < A; ++q) s = fma(T->RWP[i][q], c[q], s);
        z[i] = add_eta(et, s, z[i]);
        if (i == 0) {
          double t = T->RWP[A - 1][A - 1] * c[0];
#pragma unroll
          for (int q = 0; q < B; ++q) t = fma(T->RWP[A - 1][q], cl[q], t);
          z[i] = add_eta(etl, t, z[i]);
        }
      }
      if constexpr (!R2) {
        double f[B];
        const double* rx = jx + (k.ye + 1) * QX::RS + k.lx;
#pragma unroll
        for (int q = 0; q < B; ++q) f[q] = dot_patch<QX, A>(tw_, rx, q);
#pragma unroll
        for (int i = 0; i < B; ++i) {
          double s = 0.0;
#pragma unroll
          for (int q = 0; q < B; ++q) s = fma(T->RGP[i][q], f[q], s);
          x[i] = add_eta(et, s, x[i]);
        }
      }
    }
    if (k.below)
#pragma unroll
      for (int i = 0; i < B; ++i) { sbel[0][k.el][i] = z[i]; sbel[1][k.el][i] = R2 ? 0.0 : x[i]; }
  }
  if constexpr (!R2) {
    if (k.act && !k.w) {
      double u0[NP], u2[NP], bz[B], y[B];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        u0[q] = dot_col<NP>(tp, ue + q, NP);
        u2[q] = dot_col<NP>(tp, ue + 2 * NE * ES + q, NP);
      }
      const double l0 = dot_col<NP>(tp, ul + P, NP), l2 = dot_col<NP>(tp, ul + 2 * NE * ES + P, NP);
      double bzl = 0.0;  // the left element's B_z at x = +1
#pragma unroll
      for (int q = 0; q < B; ++q) {
        bz[q] = dot_patch<PZ, B>(tv, ze, q);
        bzl = fma(T->I_V_W[A - 1][q], dot_patch<PZ, B>(tv, ze - 1, q), bzl);
      }
      const double* xr = sx + (k.ly + 1) * PX::RS + k.j * PX::PITCH + k.lx;
#pragma unroll
      for (int i = 0; i < B; ++i) {
        double ux = 0.0, uz = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < NP; ++q) { ux = fma(T->I_P_W[i][q], u0[q], ux); uz = fma(T->I_P_W[i][q], u2[q], uz); }
#pragma unroll
        for (int q = 0; q < B; ++q) b = fma(T->I_V_W[i][q], bz[q], b);
        y[i] = -(uz * xr[PX::at(i)] - ux * b);
        if (i == 0) y[i] = 0.5 * (y[i] - (l2 * xr[PX::at(i)] - l0 * bzl));
      }
      if (res) {
        double tw_[B];
#pragma unroll
        for (int q = 0; q < B; ++q) tw_[q] = T->RGP[k.j][q];
        const double* r = jy + k.ly * QY::RS + k.lx + 1;
        double c[A], cl[B];
#pragma unroll
        for (int q = 0; q < A; ++q) c[q] = dot_patch<QY, B>(tw_, r, q);
#pragma unroll
        for (int q = 0; q < B; ++q) cl[q] = dot_patch<QY, B>(tw_, r - 1, q);
#pragma unroll
        for (int i = 0; i < B; ++i) {
          double s = 0.0;
#pragma unroll
          for (int q = 0; q < A; ++q) s = fma(T->RWP[i][q], c[q], s);
          y[i] = add_eta(et, s, y[i]);
          if (i == 0) {
            double t = T->RWP[A - 1][A - 1] * c[0];
#pragma unroll
            for (int q = 0; q < B; ++q) t = fma(T->RWP[A - 1][q], cl[q], t);
            y[i] = add_eta(etl, t, y[i]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < B; ++i) Ey[(long)gy * NXg + gx + i] = y[i];
    }
  }
  __syncthreads();
  if (k.act && k.w && !k.below) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const long g = (long)gy * NXg + gx + i;
      Ez[g] = k.j == 0 ? z[i] + sbel[0][k.el][i] : z[i];
      if (!R2) Ex[g] = k.j == 0 ? x[i] + sbel[1][k.el][i] : x[i];
    }
  }
}

template <int M, bool R2, int S>
__global__ __launch_bounds__((RT<M, R2, S>::BS)) void k_J(const double* __restrict__ Bx, const double* __restrict__ By,
                                                 const double* __restrict__ Bz, double* __restrict__ Jx,
                                                 double* __restrict__ Jy, double* __restrict__ Jz,
                                                 const MagTab* __restrict__ T, MeshP mp) {
  J_body<M, R2, S>(Bx, By, Bz, Jx, Jy, Jz, T, mp, (int)xcd_block());
}

struct J_args {
  const double* Bx;
  const double* By;
  const double* Bz;
  double* Jx;
  double* Jy;
  double* Jz;
  const MagTab* T;
  MeshP mp;
};

template <int M, bool R2, int S>
__global__ __launch_bounds__((RT<M, R2, S>::BS)) void k_J_rt(const J_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const J_args& a = A[r];
  J_body<M, R2, S>(gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.Jx), gl(a.Jy), gl(a.Jz), gl(a.T), a.mp, (int)blockIdx.x - boff[r]);
}

template <int P, int M, bool R2, int S>
__global__ __launch_bounds__((RT<M, R2, S>::BS)) void k_E(const double* __restrict__ u, const double* __restrict__ Bx,
                                                 const double* __restrict__ By, const double* __restrict__ Bz,
                                                 const double* __restrict__ Jx, const double* __restrict__ Jy,
                                                 const double* __restrict__ Jz, const double* __restrict__ eta,
                                                 double* __restrict__ Ex, double* __restrict__ Ey,
                                                 double* __restrict__ Ez, const MagTab* __restrict__ T, MeshP mp) {
  E_body<P, M, R2, S>(u, Bx, By, Bz, Jx, Jy, Jz, eta, Ex, Ey, Ez, T, mp, (int)xcd_block());
}

struct E_args {
  const double* u;
  const double* Bx;
  const double* By;
  const double* Bz;
  const double* Jx;
  const double* Jy;
  const double* Jz;
  const double* eta;
  double* Ex;
  double* Ey;
  double* Ez;
  const MagTab* T;
  MeshP mp;
};

template <int P, int M, bool R2, int S>
__global__ __launch_bounds__((RT<M, R2, S>::BS)) void k_E_rt(const E_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const E_args& a = A[r];
  E_body<P, M, R2, S>(gl(a.u), gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.Jx), gl(a.Jy), gl(a.Jz), gl(a.eta), gl(a.Ex), gl(a.Ey), gl(a.Ez), gl(a.T), a.mp, (int)blockIdx.x - boff[r]);
}

// ---------------------------------------------------------------------------------------------
// Curl update, Lorentz transpose and Ohmic heating (eq. magnetic-dae with J, E eliminated).
// MODE 0: write L_M.  MODE 1: write the SSP stage (ca*Y^n + cb*Y_s) + cb*tau*L_M(Y_s).
// ---------------------------------------------------------------------------------------------

// One thread per node, EB elements per block.  Bound by the latency of its loads and barriers: the block's
// tables and all node values are loaded before the first is stored to LDS (a table at a time and in loops per
// array, each waited for its loads: 1.35 -> 1.06 ms at 1024^2, N = 4, k = 3 (4.5 GB); 44 -> 35 us at 256^2,
// N = k = 2; 92 -> 81 us at 241 x 137, N = 5, k = 4; 200 -> 187 us at 512^2, N = 4, 2D2V).
// (the 2D2V variants up to N = 4 fit 72 VGPRs, i.e. 7 waves per SIMD, without spills; the bound
// keeps the compiler there)
template <int P, int M, int MODE, int BS, bool R2>
__device__ __forceinline__ void mag_update_body(MagIO io, const MagTab* __restrict__ T, MeshP mp, long blk) {
  using C = MC<P, M, BS>;
  constexpr int NP = C::NP, NN = C::NN, A = C::A, B = C::B, AA = C::AA, AB = C::AB, BB = C::BB, EB = C::EB,
                NT = C::NT;
  __shared__ double sbx[EB][AB], sby[EB][AB], sbz[EB][BB];
  __shared__ double sex[EB][AB], sey[EB][AB], sez[EB][AA];
  __shared__ double sjx[EB][AB], sjy[EB][AB], sjz[EB][AA];
  // Lorentz loads at the auxiliary nodes, one buffer per element: fz (W nodes, x and y parts), fx
  // (N_x nodes, y and z parts), fy (N_y nodes, x and z parts).  After a barrier the new velocities
  // for the closing element statistics reuse it, which keeps the block's LDS within five blocks
  // per CU at N = 4.
  constexpr int NF = 2 * AA + 4 * AB;
  static_assert(3 * NN <= NF, "the velocity buffer must fit in the Lorentz-load buffer");
  __shared__ double sf[EB][NF];
  constexpr UpdTab o(P, M);
  __shared__ double tb[o.n];
  auto *const tDWG = (const double(*)[A])(tb + o.DWG), *const tDWV = (const double(*)[A])(tb + o.DWV);
  auto *const tIGV = (const double(*)[B])(tb + o.IGV), *const tIGW = (const double(*)[B])(tb + o.IGW);
  auto *const tIVG = (const double(*)[B])(tb + o.IVG), *const tIVW = (const double(*)[B])(tb + o.IVW);
  auto *const tIPW = (const double(*)[NP])(tb + o.IPW), *const tIPG = (const double(*)[NP])(tb + o.IPG);
  auto *const tIGP = (const double(*)[B])(tb + o.IGP);
  auto *const tIWP = (const double(*)[A])(tb + o.IWP);
  const double *const tww = tb + o.ww, *const twg = tb + o.wg, *const twp = tb + o.wp;
  const int tid = threadIdx.x, el = tid / NT, t = tid - el * NT;
  const long e = blk * EB + el;
  const bool act = el < EB && e < mp.K;
  long ex, ey;
  elem_xy(mp, act ? e : 0, ex, ey);
  const long KN = mp.K * NN;
  double* const fz = sf[act ? el : 0];
  double* const fx = fz + 2 * AA;
  double* const fy = fx + 2 * AB;
  constexpr int NTB = (o.n + BS - 1) / BS;
  double vt[NTB];
#pragma unroll
  for (int k = 0; k < NTB; ++k) vt[k] = tid + k * BS < o.n ? T->upd[tid + k * BS] : 0.0;
  // values used only at the end are loaded first, so that their latency overlaps the work
  // (MODE 1 keeps only y0 = ca*Y^n + cb*Y_s of every value and adds cb*tau*L_M at the end, so
  // that one register pair per value stays live across the kernel instead of two)
  double rq = 1.0, et = 0.0, y0[4] = {0, 0, 0, 0}, b0[3] = {0, 0, 0};
  long gown = 0;
  if (act && t < NN) {
    const long n = e * NN + t;
    rq = io.rho[n];
    et = io.eta ? io.eta[e] : 0.0;
    if (MODE == 1) {
#pragma unroll
      for (int d = 0; d < (R2 ? 2 : 3); ++d) y0[d] = io.ca * io.un[d * KN + n] + io.cb * io.us[d * KN + n];
      y0[3] = io.ca * io.en[n] + io.cb * io.es[n];
    }
  }
  if (act && t < BB) {
    gown = gix(mp, B, ex, ey, t % B, t / B);
    if (MODE == 1) {
      b0[0] = io.ca * io.bxn[gown] + io.cb * io.bxs[gown];
      b0[1] = io.ca * io.byn[gown] + io.cb * io.bys[gown];
      if (!R2) b0[2] = io.ca * io.bzn[gown] + io.cb * io.bzs[gown];
    }
  }
  // the element's B, E and J nodes (one of each kind per thread): all loads are issued before the first is stored
  {
    const long G = (long)mp.nx * B * mp.ny * B;
    const int NXg = mp.nx * B, NYg = mp.ny * B, x0 = (int)ex * B, y0_ = (int)ey * B;
    auto off = [&](int i, int j) {
      const int gx = x0 + i, gy = y0_ + j;
      return (unsigned)((gy >= NYg ? gy - NYg : gy) * NXg + (gx >= NXg ? gx - NXg : gx)) * 8u;
    };
    double vbx = 0.0, vby = 0.0, vbz = 0.0, vex = 0.0, vey = 0.0, vez = 0.0, vjx = 0.0, vjy = 0.0, vjz = 0.0;
    if (act && t < AB) {
      const unsigned nx_ = off(t % B, t / B), ny_ = off(t % A, t / A);  // N_x and N_y nodes
      vbx = bld(node_rsrc(io.bxs, G), ny_);
      vby = bld(node_rsrc(io.bys, G), nx_);
      if (!R2) {  // in-plane E and J (none in the 2D2V system)
        vex = bld(node_rsrc(io.ex, G), nx_);
        vjx = bld(node_rsrc(io.jx, G), nx_);
        vey = bld(node_rsrc(io.ey, G), ny_);
        vjy = bld(node_rsrc(io.jy, G), ny_);
      }
    }
    if (act && t < AA) {
      const unsigned w = off(t % A, t / A);
      vez = bld(node_rsrc(io.ez, G), w);
      vjz = bld(node_rsrc(io.jz, G), w);
    }
    if (!R2 && act && t < BB) vbz = bld(node_rsrc(io.bzs, G), (unsigned)gown * 8u);
#pragma unroll
    for (int k = 0; k < NTB; ++k)
      if (tid + k * BS < o.n) tb[tid + k * BS] = vt[k];
    if (act && t < AB) {
      sbx[el][t] = vbx; sby[el][t] = vby;
      if (!R2) { sex[el][t] = vex; sjx[el][t] = vjx; sey[el][t] = vey; sjy[el][t] = vjy; }
    }
    if (act && t < AA) { sez[el][t] = vez; sjz[el][t] = vjz; }
    if (!R2 && act && t < BB) sbz[el][t] = vbz;
  }
  __syncthreads();
  if (act && t < BB) {  // strong curl at the element's owned B nodes
    const int i = t % B, j = t / B;
    const long g = gown;
    double dbx = 0.0, dby = 0.0;
#pragma unroll
    for (int k = 0; k < A; ++k) {
      dbx += tDWG[j][k] * sez[el][k * A + i];
      dby += tDWG[i][k] * sez[el][j * A + k];
    }
    dbx *= -(2.0 * mp.rhy);
    dby *= (2.0 * mp.rhx);
    double dxey = 0.0, dyex = 0.0;
    if constexpr (!R2) {
#pragma unroll
    for (int l = 0; l < B; ++l) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < A; ++k) s += tDWV[i][k] * sey[el][l * A + k];
      dxey += tIGV[j][l] * s;
    }
#pragma unroll
    for (int l = 0; l < A; ++l) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < B; ++k) s += tIGV[i][k] * sex[el][l * B + k];
      dyex += tDWV[j][l] * s;
    }
    }
    const double dbz = R2 ? 0.0 : -((2.0 * mp.rhx) * dxey - (2.0 * mp.rhy) * dyex);
    if (MODE == 0) {
      io.obx[g] = dbx; io.oby[g] = dby; io.obz[g] = dbz;
    } else {
      const double ct = io.cb * io.tau;
      io.obx[g] = b0[0] + ct * dbx;
      io.oby[g] = b0[1] + ct * dby;
      io.obz[g] = R2 ? 0.0 : b0[2] + ct * dbz;
    }
  }
  // weighted Lorentz loads f_a at the auxiliary nodes (transpose of the coupling form)
  if (act && t < AA) {
    const int i = t % A, j = t / A;
    double bxv = 0.0, byv = 0.0;
#pragma unroll
    for (int k = 0; k < B; ++k) {
      bxv += tIGW[j][k] * sbx[el][k * A + i];
      byv += tIGW[i][k] * sby[el][j * B + k];
    }
    const double w = mp.J * tww[i] * tww[j] * sjz[el][t];
    fz[t] = -byv * w;      // x
    fz[AA + t] = bxv * w;  // y
  }
  if (!R2 && act && t < AB) {
    {
      const int i = t % B, j = t / B;  // N_x node: (0, -B_z J_x, B_y J_x)
      double bzv = 0.0;
#pragma unroll
      for (int jj = 0; jj < B; ++jj) {
        double s = 0.0;
#pragma unroll
        for (int ii = 0; ii < B; ++ii) s += tIVG[i][ii] * sbz[el][jj * B + ii];
        bzv += tIVW[j][jj] * s;
      }
      const double w = mp.J * twg[i] * tww[j] * sjx[el][t];
      fx[t] = -bzv * w;             // y
      fx[AB + t] = sby[el][t] * w;  // z
    }
    {
      const int i = t % A, j = t / A;  // N_y node: (B_z J_y, 0, -B_x J_y)
      double bzv = 0.0;
#pragma unroll
      for (int jj = 0; jj < B; ++jj) {
        double s = 0.0;
#pragma unroll
        for (int ii = 0; ii < B; ++ii) s += tIVW[i][ii] * sbz[el][jj * B + ii];
        bzv += tIVG[j][jj] * s;
      }
      const double w = mp.J * tww[i] * twg[j] * sjy[el][t];
      fy[t] = bzv * w;               // x
      fy[AB + t] = -sbx[el][t] * w;  // z
    }
  }
  __syncthreads();
  const bool node = act && t < NN;
  double vnew[3] = {0.0, 0.0, 0.0};
  if (node) {
    const int qi = t % NP, qj = t / NP;
    // transpose of the interpolation to the auxiliary nodes, factorised over the two directions
    double du[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int j = 0; j < A; ++j) {
      double s0 = 0.0, s1 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
      for (int i = 0; i < A; ++i) {
        const double I = tIPW[i][qi];
        s0 += I * fz[j * A + i];
        s1 += I * fz[AA + j * A + i];
      }
      if constexpr (!R2) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
          const double I = tIPG[i][qi];
          t1 += I * fx[j * B + i];
          t2 += I * fx[AB + j * B + i];
        }
      }
      const double Iy = tIPW[j][qj];
      du[0] += Iy * s0;
      du[1] += Iy * (s1 + t1);
      du[2] += Iy * t2;
    }
#pragma unroll 1
    for (int j = 0; !R2 && j < B; ++j) {
      double s0 = 0.0, s2 = 0.0;
#pragma unroll
      for (int i = 0; i < A; ++i) {
        const double I = tIPW[i][qi];
        s0 += I * fy[j * A + i];
        s2 += I * fy[AB + j * A + i];
      }
      const double Iy = tIPG[j][qj];
      du[0] += Iy * s0;
      du[2] += Iy * s2;
    }
    const long n = e * NN + t;
    const double Mq = mp.J * twp[qi] * twp[qj];
    double de = 0.0;
    if (et != 0.0) {
      double jx = 0.0, jy = 0.0, jz = 0.0;
      if constexpr (!R2) {
#pragma unroll
        for (int j = 0; j < A; ++j) {
          double s = 0.0;
#pragma unroll
          for (int i = 0; i < B; ++i) s += tIGP[qi][i] * sjx[el][j * B + i];
          jx += tIWP[qj][j] * s;
        }
#pragma unroll
        for (int j = 0; j < B; ++j) {
          double s = 0.0;
#pragma unroll
          for (int i = 0; i < A; ++i) s += tIWP[qi][i] * sjy[el][j * A + i];
          jy += tIGP[qj][j] * s;
        }
      }
#pragma unroll
      for (int j = 0; j < A; ++j) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < A; ++i) s += tIWP[qi][i] * sjz[el][j * A + i];
        jz += tIWP[qj][j] * s;
      }
      de = et * (jx * jx + jy * jy + jz * jz) * rcp_refined(rq);  // rho > 0
    }
    // (the 2D2V system writes u_z = 0, so that no stage buffer carries a stale value)
    const double irm = rcp_refined(rq * Mq);  // 1 / (rho M), both positive
    if (MODE == 0) {
      for (int d = 0; d < 3; ++d) io.ou[d * KN + n] = (R2 && d == 2) ? 0.0 : du[d] * irm;
      io.oe[n] = de;
    } else {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double v = (R2 && d == 2) ? 0.0 : y0[d] + (io.cb * io.tau) * (du[d] * irm);
        io.ou[d * KN + n] = v;
        vnew[d] = v;
      }
      io.oe[n] = y0[3] + (io.cb * io.tau) * de;
    }
  }
  if (MODE == 1 && io.ustats) {
    // element statistics of the new velocity (GLL-weighted sum, min, max), as the velocity-OE
    // sensor needs them
    __syncthreads();  // every lane has finished reading the Lorentz loads
    if (node)
#pragma unroll
      for (int d = 0; d < 3; ++d) fz[d * NN + t] = vnew[d];
    __syncthreads();
    constexpr int NU = R2 ? 2 : 3;  // statistics [K][NU][3] of the carried components
    for (int tk = t; act && tk < 3 * NU; tk += NT) {
      const int c = tk / 3, kind = tk - 3 * c;
      double sm = 0.0, mn = DBL_MAX, mx = -DBL_MAX;
      for (int k = 0; k < NN; ++k) {
        const double v = fz[c * NN + k];
        sm += (twp[k % NP] * twp[k / NP]) * v;
        mn = fmin(mn, v); mx = fmax(mx, v);
      }
      io.ustats[(e * NU + c) * 3 + kind] = kind == 0 ? sm : (kind == 1 ? mn : mx);
    }
  }
}

template <int P, int M, int MODE, int BS, bool R2>
__global__ __launch_bounds__(BS, (R2 && P <= 4) ? 7 : 1) void k_mag_update(MagIO io, const MagTab* __restrict__ T, MeshP mp) {
  mag_update_body<P, M, MODE, BS, R2>(io, T, mp, xcd_block());
}

using ::gl;
// a MagIO read from a run-table argument struct, its pointers loaded as global-memory pointers
__device__ __forceinline__ MagIO gl(const MagIO& s) {
  MagIO o = s;
  o.rho = gl(s.rho); o.us = gl(s.us); o.es = gl(s.es); o.bxs = gl(s.bxs); o.bys = gl(s.bys); o.bzs = gl(s.bzs);
  o.un = gl(s.un); o.en = gl(s.en); o.bxn = gl(s.bxn); o.byn = gl(s.byn); o.bzn = gl(s.bzn);
  o.jx = gl(s.jx); o.jy = gl(s.jy); o.jz = gl(s.jz); o.ex = gl(s.ex); o.ey = gl(s.ey); o.ez = gl(s.ez);
  o.eta = gl(s.eta);
  o.oe = gl(s.oe); o.ou = gl(s.ou); o.obx = gl(s.obx); o.oby = gl(s.oby); o.obz = gl(s.obz);
  o.ustats = gl(s.ustats);
  return o;
}

struct mag_update_args {
  MagIO io;
  const MagTab* T;
  MeshP mp;
};

template <int P, int M, int MODE, int BS, bool R2>
__global__ __launch_bounds__(BS, (R2 && P <= 4) ? 7 : 1) void k_mag_update_rt(const mag_update_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const mag_update_args& a = A[r];
  mag_update_body<P, M, MODE, BS, R2>(gl(a.io), gl(a.T), a.mp, (long)blockIdx.x - boff[r]);
}

// per-element statistics of NC nodal fields [NC][K][NN] -> [K][NC][3] (GLL-weighted sum, min, max)
template <int P, int NC>
__global__ __launch_bounds__(256) void k_field_stats(const double* __restrict__ f, double* __restrict__ stats,
                                                     const MagTab* __restrict__ T, MeshP mp) {
  constexpr int NP = P + 1, NN = NP * NP, EB = 256 / NN;
  __shared__ double sv[NC][EB * NN];
  const int tid = threadIdx.x, el = tid / NN, q = tid - el * NN;
  const long e = (long)blockIdx.x * EB + el;
  const bool act = el < EB && e < mp.K;
  const long KN = mp.K * NN;
  if (act)
    for (int c = 0; c < NC; ++c) sv[c][tid] = f[c * KN + e * NN + q];
  __syncthreads();
  for (int tk = q; act && tk < NC * 3; tk += NN) {
    const int c = tk / 3, kind = tk - 3 * c;
    double s = 0.0, mn = DBL_MAX, mx = -DBL_MAX;
    for (int k = 0; k < NN; ++k) {
      const double v = sv[c][el * NN + k];
      s += (T->wp[k % NP] * T->wp[k / NP]) * v;
      mn = fmin(mn, v); mx = fmax(mx, v);
    }
    stats[(e * NC + c) * 3 + kind] = kind == 0 ? s : (kind == 1 ? mn : mx);
  }
}

// ---------------------------------------------------------------------------------------------
// Velocity OE (eq. magnetic-oe-sensor .. eq. magnetic-oe-map).  The rho-weighted projections use
// the shell-ordered tensor Legendre basis orthonormalised in the rho-weighted product,
// psi = phi L^{-T} with G = L L^T the Gram matrix.  rho is frozen during a magnetic substep, so
// Psi[q][k] = psi_k(x_q) is computed once per substep (k_vel_prep) and reused by the three stages: per stage k_vel_sensor forms the
// damping factors and k_vel_proj applies the map.
// ---------------------------------------------------------------------------------------------
// shell index of mode k in the shell ordering (shell l holds modes l^2 .. (l+1)^2 - 1)
__host__ __device__ constexpr int shell_of(int k) {
  int l = 0;
  while ((l + 1) * (l + 1) <= k) ++l;
  return l;
}

// shell-ordered tensor Legendre mode k -> (a, b): shell l = max(a, b) holds modes l^2 .. (l+1)^2 - 1,
// (a, l) for a < l first, then (l, b) for b = 0..l (the order of the basis tables)
__host__ __device__ constexpr int mode_a(int k) {
  const int l = shell_of(k), r = k - l * l;
  return r < l ? r : l;
}
__host__ __device__ constexpr int mode_b(int k) {
  const int l = shell_of(k), r = k - l * l;
  return r < l ? l : r - l;
}

// threads per block of the velocity-OE preparation (EB = MHD_PREP_BS / (N+1)^2 elements a block)
#ifndef MHD_PREP_BS
#define MHD_PREP_BS 256
#endif
template <int P>
struct VP {
  static constexpr int NP = P + 1, NN = NP * NP, NK = psi_modes(P), EB = MHD_PREP_BS / NN;
};

// The basis is needed for the shells 0..p-1 only: they span Q^{p-1}, and since the projection onto all
// of Q^p is the identity, the last shell's part of a field is the field minus the others' parts.  So
// the Gram matrix, its Cholesky factor and the table hold NK = p^2 modes instead of (p+1)^2.
//
// EB elements per block.  The node weights and the substitution run with one thread per node, the
// factorisation with one thread per (element, row), packed onto the block's first EB NK threads, so
// that its lanes are full and the other waves only pass the barriers.  The Gram matrix is formed by
// sum factorisation and packed in LDS; a left-looking Cholesky (one barrier per column) overwrites it
// with L, and row q of Psi = Phi L^{-T} follows by forward substitution with L read from LDS.  Mode
// indices are compile-time constants in the unrolled loops, and masked arithmetic replaces branches;
// the Cholesky dot products run on two accumulators to halve their FMA chains.
template <int P>
__device__ __forceinline__ void vel_prep_body(const double* __restrict__ rho, double* __restrict__ Psi,
                                                 const HydroTab* __restrict__ H, MeshP mp, long blk) {
  using C = VP<P>;
  constexpr int NP = C::NP, NN = C::NN, NK = C::NK, EB = C::EB;
  // packed triangle, padded to an odd stride: the elements of a wave read the same entry of their own
  // triangles from different banks
  constexpr int NL = (NK * (NK + 1) / 2) | 1;
  constexpr int NPS = P * (P + 1) / 2;  // pairs a <= a' of the x modes 0..p-1
  // sH holds the line partials Hm[qj][a][a'] for a <= a', and then the pivot reciprocals srd (first
  // written after the barrier that follows the last reads of the partials).  Masked lanes store to
  // one of eight dummy slots.
  constexpr int NH = NP * NPS > NK ? NP * NPS : NK;
  __shared__ double sL[EB * NL], sH[EB * NH], sw[EB * NN], sV[NP][NP], sdum[8];
  const int tid = threadIdx.x;
  const long e0 = blk * EB;
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;  // elements of this block
  for (int t = tid; t < NP * NP; t += MHD_PREP_BS) sV[t / NP][t % NP] = H->V[t / NP][t % NP];
  if (tid < nel * NN) {
    const int q = tid % NN;
    sw[tid] = mp.J * H->w[q % NP] * H->w[q / NP] * rho[e0 * NN + tid];
  }
  __syncthreads();
  // sum factorisation: Hm[qj][a][a'] = sum_qi W[qj][qi] V[qi][a] V[qi][a'], symmetric in (a, a'),
  // kept for a <= a' (entry p of a line runs over (0, 0..P-1), (1, 1..P-1), ...)
  for (int t = tid; t < nel * NP * NPS; t += MHD_PREP_BS) {
    const int line = t / NPS;  // element * NP + qj
    int p = t - line * NPS, a = 0;
    while (p >= P - a) { p -= P - a; ++a; }
    const int a2 = a + p;
    double s = 0.0;
#pragma unroll
    for (int ii = 0; ii < NP; ++ii) s += sw[line * NP + ii] * sV[ii][a] * sV[ii][a2];
    sH[(line / NP) * NH + (line % NP) * NPS + (t - line * NPS)] = s;
  }
  __syncthreads();
  {
    const bool row = tid < nel * NK;  // this thread owns row q of element el
    const int el = row ? tid / NK : 0, q = row ? tid - el * NK : 0;  // the others shadow row 0
    double* const L = sL + el * NL;
    double* const srd = sH + el * NH;
    // (LDS stores below go through address selects, not branches: a lane that must not write
    // targets its own dummy slot)
    // Gram row q (shell order): G[q][k'] = sum_qj V[qj][b'] (V[qj][b] Hm[qj][a][a']), k' <= q,
    // packed; row q starts at rq = q (q + 1) / 2
    const int rq = q * (q + 1) / 2;
    double Lr[NK];
    double piv = 1.0;
    if (tid < EB * NK) {  // whole waves past the rows skip the arithmetic
      const int l = [&] { int s = 0; while ((s + 1) * (s + 1) <= q) ++s; return s; }();
      const int ka = q - l * l < l ? q - l * l : l, kb = q - l * l < l ? l : q - l * l - l;
      int hx[P];  // position of the pair (min(a_q, a'), max(a_q, a')) in a line of sH
#pragma unroll
      for (int a2 = 0; a2 < P; ++a2) {
        const int lo = ka < a2 ? ka : a2, hi = ka < a2 ? a2 : ka;
        hx[a2] = lo * P - lo * (lo - 1) / 2 + (hi - lo);
      }
      double w[NP][P];
#pragma unroll
      for (int jj = 0; jj < NP; ++jj)
#pragma unroll
        for (int a2 = 0; a2 < P; ++a2) w[jj][a2] = sV[jj][kb] * sH[el * NH + jj * NPS + hx[a2]];
#pragma unroll
      for (int k2 = 0; k2 < NK; ++k2) {
        double s = 0.0;
#pragma unroll
        for (int jj = 0; jj < NP; ++jj) s += H->V[jj][mode_b(k2)] * w[jj][mode_a(k2)];  // uniform: scalar loads
        Lr[k2] = s;              // the row of G, kept in registers
        if (k2 == q) piv = s;    // G[q][q]
      }
    }
    __syncthreads();  // every lane has read the partials, whose space the pivot reciprocals take
    // Left-looking Cholesky G = L L^T, one column per step.  Thread q keeps its row of L in registers.
    // At step k the threads q > k form L[q][k] = (G[q][k] - sum_{m<k} L[q][m] L[k][m]) / L[k][k] with
    // row k read from LDS, and the thread of row k + 1, whose row is then complete up to the diagonal,
    // forms its pivot from its running G[q][q] - sum_m L[q][m]^2.  srd[k] = 1 / L[k][k].
    {
      const double rk = rsqrt_refined(piv);  // used by row 0 only
      *((row && q == 0) ? &L[0] : &sdum[tid & 7]) = piv * rk;
      *((row && q == 0) ? &srd[0] : &sdum[tid & 7]) = rk;
    }
    __syncthreads();
    // Only the rows q > k read row k; the lanes at or above the diagonal stay masked (measured
    // faster than letting them read and discard).
#pragma unroll
    for (int k = 0; k + 1 < NK; ++k) {
      if (tid < EB * NK) {
        if (q > k) {
          double s0 = Lr[k], s1 = 0.0;  // G[q][k]
#pragma unroll
          for (int m = 0; m < k; ++m) {
            if (m & 1) s1 -= Lr[m] * L[k * (k + 1) / 2 + m];
            else s0 -= Lr[m] * L[k * (k + 1) / 2 + m];
          }
          Lr[k] = (s0 + s1) * srd[k];  // L[q][k]
        }
        *((row && q > k) ? &L[rq + k] : &sdum[tid & 7]) = Lr[k];
        piv -= Lr[k] * Lr[k];
        const double rk = rsqrt_refined(piv);  // pivot of row k + 1 (used by that row only)
        *((row && q == k + 1) ? &L[rq + q] : &sdum[tid & 7]) = piv * rk;
        *((row && q == k + 1) ? &srd[k + 1] : &sdum[tid & 7]) = rk;
      }
      __syncthreads();
    }
  }
  // row q of Psi = Phi L^{-T}: forward substitution over the modes with the row in registers
  // (L is read from LDS as broadcasts); Phi[q][k] = V[qi][a_k] V[qj][b_k]
  if (tid >= nel * NN) return;
  const int el = tid / NN, q = tid - el * NN, qi = q % NP, qj = q / NP;
  const double* const L = sL + el * NL;
  const double* const srd = sH + el * NH;
  double vi[P], vj[P];
#pragma unroll
  for (int a = 0; a < P; ++a) { vi[a] = sV[qi][a]; vj[a] = sV[qj][a]; }
  // Right-looking order: once psi[k] is final, L[j][k] psi[k] is subtracted from every later
  // entry j.  Each entry receives the same subtractions in the same order as in the row-by-row
  // form, but the entries are independent chains.
  double psi[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) psi[k] = vi[mode_a(k)] * vj[mode_b(k)];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    psi[k] *= srd[k];
#pragma unroll
    for (int j = k + 1; j < NK; ++j) psi[j] -= L[j * (j + 1) / 2 + k] * psi[k];
  }
  // row q of the element's table, stored directly (rows are 16-byte aligned: psi_row is even)
  constexpr long PS = psi_stride(P), RS = psi_row(P);
  double2* out = reinterpret_cast<double2*>(Psi + (e0 + el) * PS + q * RS);
#pragma unroll
  for (int k2 = 0; k2 < NK / 2; ++k2) out[k2] = double2{psi[2 * k2], psi[2 * k2 + 1]};
  if (NK % 2) out[NK / 2] = double2{psi[NK - 1], 0.0};
}

template <int P>
__global__ __launch_bounds__(MHD_PREP_BS) void k_vel_prep(const double* __restrict__ rho, double* __restrict__ Psi,
                                                 const HydroTab* __restrict__ H, MeshP mp) {
  vel_prep_body<P>(rho, Psi, H, mp, (long)blockIdx.x);
}

struct vel_prep_args {
  const double* rho;
  double* Psi;
  const HydroTab* H;
  MeshP mp;
};

template <int P>
__global__ __launch_bounds__(MHD_PREP_BS) void k_vel_prep_rt(const vel_prep_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const vel_prep_args& a = A[r];
  vel_prep_body<P>(gl(a.rho), gl(a.Psi), gl(a.H), a.mp, (long)blockIdx.x - boff[r]);
}

// Tile of the velocity-OE sensor: TX x TY elements and the ring around them.  One thread per component and
// face, the tile's (TX + 1) TY x faces on the block's first half, its TX (TY + 1) y faces on the second, so that
// a wave has one direction.  The wave speeds are row tasks, one GLL row of an element each.  5 x 5 elements
// leave three blocks per CU at N = 4; 6 x 6 fill more lanes but leave two (0.56 against 0.52 ms at 1024^2).  S: tile
// shape as RT's, the row's and column's length for as many staged elements (65536 x 1: N = 4 56 us against 199, N = 6
// 137 against 550).
template <int P, int M, bool R2, int S>
struct VS {
  static constexpr int NP = P + 1, NN = NP * NP, ES = NN | 1;  // odd element stride in LDS: no bank conflicts
  static constexpr int A = M + 2, B = M + 1, BS = 256, NU = R2 ? 2 : 3;  // u_z = 0 in the 2D2V system
  static constexpr int TL = P < 6 ? 15 : 12;
  static constexpr int TX = S == 0 ? 5 : (S == 1 ? TL : 1), TY = S == 0 ? (P < 6 ? 5 : 4) : (S == 1 ? 1 : TL), TE = TX * TY;
  static constexpr int NX = (TX + 1) * TY, NY = TX * (TY + 1);  // faces
  static constexpr int NS = TE + 2 * (TX + TY);                 // staged elements: the tile's, then the ring's
  static_assert(NU * NX <= BS / 2 && NU * NY <= BS / 2, "a thread per component and face");
};

// Velocity-OE sensor (eq. magnetic-oe-sensor, eq. magnetic-oe-rate, eq. magnetic-oe-factor): the element's
// damping factors D_l (l = 0..p), Dfac[K][p+1].  Every face's jumps are formed once per tile from LDS.  u is
// only read here (the projection kernel that updates it runs afterwards).  Measured, against a thread per
// node with the neighbours staged per element: 0.98 -> 0.52 ms at 1024^2, N = 4, k = 3 (1.31 GB), 61 -> 37 us
// at 241 x 137, N = 5, 32 -> 17 us at 256^2, N = 2.  Bound by VALU issue and the latency of its staging loads.
template <int P, int M, bool R2, int S>
__device__ __forceinline__ void vel_sensor_body(const double* __restrict__ rho, const double* __restrict__ u,
                                                    const double* __restrict__ Bx, const double* __restrict__ By,
                                                    const double* __restrict__ Bz, const double* __restrict__ lines,
                                                    const double* __restrict__ glob, double* __restrict__ Dfac,
                                                    const HydroTab* __restrict__ H, const MagTab* __restrict__ T,
                                                    const MeshP& mp, double tau, double sM, int blk) {
  using C = VS<P, M, R2, S>;
  constexpr int NP = C::NP, NN = C::NN, ES = C::ES, A = C::A, B = C::B, BS = C::BS, NU = C::NU;
  constexpr int TX = C::TX, TY = C::TY, TE = C::TE, NS = C::NS, NX = C::NX, NY = C::NY;
  using PX = Patch<TY * B, TX * B + 1, B, TX, BS>;
  using PY = Patch<TY * B + 1, TX * B, B, TX, BS>;
  using PZ = Patch<TY * B, TX * B, B, TX, BS>;
  // su[c][staged element][ES]; then the faces' jumps sj[c][face][NP] (x faces first)
  constexpr int NUS = NU * NS * ES, NJ = NU * (NX + NY) * NP;
  __shared__ double su[NUS > NJ ? NUS : NJ], sr[TE * ES], sx[PX::SIZE], sy[PY::SIZE], sz[R2 ? 1 : PZ::SIZE];
  __shared__ double sws[2][NP][TE], ssg[TE][2 * NP], samp[2][TX > TY ? TX : TY];
  const int tid = threadIdx.x;
  int tx0, ty0;
  tile_of(blk, (mp.nx + TX - 1) / TX, (mp.ny + TY - 1) / TY, tx0, ty0);
  tx0 *= TX; ty0 *= TY;
  const int tw = mp.nx - tx0 < TX ? mp.nx - tx0 : TX, th = mp.ny - ty0 < TY ? mp.ny - ty0 : TY;
  const long KN = mp.K * NN;
  // the nodes of the staged elements (ring: left, right column, bottom, top row), coalesced
  constexpr int NR = (NS * NN + BS - 1) / BS, NRR = (TE * NN + BS - 1) / BS;
  {
    double v[NR][NU], w[NRR];
    int slot[NR];
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int n = tid + m * BS, s = n / NN, q = n - s * NN;
      int x, y;
      bool in;
      if (s < TE) { y = s / TX; x = s - y * TX; in = x < tw && y < th; }
      else if (s < TE + 2 * TY) { const int h = s - TE; x = h < TY ? -1 : tw; y = h < TY ? h : h - TY; in = y < th; }
      else { const int h = s - TE - 2 * TY; y = h < TX ? -1 : th; x = h < TX ? h : h - TX; in = s < NS && x < tw; }
      slot[m] = in ? s * ES + q : -1;
      if (in) {
        const unsigned o = ((unsigned)(wrap32(ty0 + y, mp.ny) * mp.nx + wrap32(tx0 + x, mp.nx)) * NN + q) * 8u;
#pragma unroll
        for (int d = 0; d < NU; ++d) v[m][d] = bld(node_rsrc(u + d * KN, KN), o);
        if (m < NRR && s < TE) w[m < NRR ? m : 0] = bld(node_rsrc(rho, KN), o);
      }
    }
    PX px;
    PY py;
    px.load(Bx, mp, tx0 * B, ty0 * B, tw * B + 1, th * B);
    py.load(By, mp, tx0 * B, ty0 * B, tw * B, th * B + 1);
    if constexpr (!R2) {
      PZ pz;
      pz.load(Bz, mp, tx0 * B, ty0 * B, tw * B, th * B);
      pz.store(sz);
    }
#pragma unroll
    for (int m = 0; m < NR; ++m)
      if (slot[m] >= 0) {
#pragma unroll
        for (int d = 0; d < NU; ++d) su[d * NS * ES + slot[m]] = v[m][d];
        if (m < NRR && slot[m] < TE * ES) sr[slot[m]] = w[m < NRR ? m : 0];
      }
    px.store(sx);
    py.store(sy);
  }
  // cross-line amplitudes shared by the components: rows, then columns
  if (tid < TY + TX) {
    const int D = tid < TY ? 0 : 1, i = D ? tid - TY : tid;
    if (i < (D ? tw : th)) {
      const double* l = lines + (D ? mp.ny + tx0 + i : ty0 + i) * (NU * 3);
      const double rn = D ? mp.r4ny : mp.r4nx;
      double a = 0.0;
#pragma unroll
      for (int d = 0; d < NU; ++d) {
        const double gm = glob[d * 3] * mp.r4K, m = l[d * 3] * rn;
        const double dOm = fmax(glob[d * 3 + 2] - gm, gm - glob[d * 3 + 1]);
        a = fmax(a, fmax(fmax(l[d * 3 + 2] - m, m - l[d * 3 + 1]), 1e-6 * dOm));
      }
      samp[D][i] = a;
    }
  }
  __syncthreads();
  // the largest wave speeds |u_x| + c_A, |u_y| + c_A of each GLL row
  for (int k = tid; k < TE * NP; k += BS) {
    const int j = k / TE, en = k - j * TE, y = en / TX, x = en - y * TX;
    if (x < tw && y < th) {
      double b2[NP];
      {
        double c[A], t[B];
#pragma unroll
        for (int i = 0; i < B; ++i) t[i] = T->I_G_P[j][i];
#pragma unroll
        for (int i = 0; i < A; ++i) c[i] = dot_patch<PX, B>(t, sx + y * PX::RS + x, i);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          double s = 0.0;
#pragma unroll
          for (int i = 0; i < A; ++i) s = fma(T->I_W_P[q][i], c[i], s);
          b2[q] = s * s;
        }
      }
      SCHED_FENCE();
      {
        double c[B], t[A];
#pragma unroll
        for (int i = 0; i < A; ++i) t[i] = T->I_W_P[j][i];
#pragma unroll
        for (int i = 0; i < B; ++i) c[i] = dot_patch<PY, A>(t, sy + y * PY::RS + x, i);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          double s = 0.0;
#pragma unroll
          for (int i = 0; i < B; ++i) s = fma(T->I_G_P[q][i], c[i], s);
          b2[q] = fma(s, s, b2[q]);
        }
      }
      SCHED_FENCE();
      if constexpr (!R2) {
        double c[B], t[B];
#pragma unroll
        for (int i = 0; i < B; ++i) t[i] = T->I_V_P[j][i];
#pragma unroll
        for (int i = 0; i < B; ++i) c[i] = dot_patch<PZ, B>(t, sz + y * PZ::RS + x, i);
#pragma unroll
        for (int q = 0; q < NP; ++q) {
          double s = 0.0;
#pragma unroll
          for (int i = 0; i < B; ++i) s = fma(T->I_V_P[q][i], c[i], s);
          b2[q] = fma(s, s, b2[q]);
        }
      }
      SCHED_FENCE();
      double ax = 0.0, ay = 0.0;
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int n = en * ES + j * NP + q;
        const double va = sqrt(b2[q]) * rsqrt_refined(sr[n]);  // rho > 0
        ax = fmax(ax, fabs(su[n]) + va);
        ay = fmax(ay, fabs(su[NS * ES + n]) + va);
      }
      sws[0][j][en] = ax;
      sws[1][j][en] = ay;
    }
  }
  SCHED_FENCE();
  // the thread's face (x faces: fx counts the TX + 1 faces of a row) and component
  const int D = __builtin_amdgcn_readfirstlane(tid >= BS / 2 ? 1 : 0);
  const int t = tid - D * (BS / 2), nf = D ? NY : NX, c = t / nf, f = t - c * nf;
  const int fx = D ? f % TX : f % (TX + 1), fy = D ? f / TX : f / (TX + 1);
  const bool act = c < NU && (D ? fx < tw && fy <= th : fx <= tw && fy < th);
  double J[NP];
  if (act) {
    const double* sv = su + c * NS * ES;
    if (D == 0)
      face_jumps<P, 0>(sv + (fx == 0 ? TE + fy : fy * TX + fx - 1) * ES, sv + (fx == tw ? TE + TY + fy : fy * TX + fx) * ES, H, J);
    else
      face_jumps<P, 1>(sv + (fy == 0 ? TE + 2 * TY + fx : (fy - 1) * TX + fx) * ES,
                       sv + (fy == th ? TE + 2 * TY + TX + fx : fy * TX + fx) * ES, H, J);
  }
  __syncthreads();
  if (act) {
    // a component that is constant to roundoff (its nodal values agree to 2^10 ulps of the field's size, an exact
    // test) does not count
    const double gmn = glob[c * 3 + 1], gmx = glob[c * 3 + 2];
    const bool cst = gmx - gmn <= 1024.0 * EPSM * fmax(fabs(gmx), fabs(gmn));
    double* o = su + (c * (NX + NY) + (D ? NX + f : f)) * NP;
#pragma unroll
    for (int r = 0; r < NP; ++r) o[r] = cst ? 0.0 : J[r];
  }
  __syncthreads();
  // sigma^u: the two faces' jumps, maximum over the components, against the shared amplitude
  for (int k = tid; k < TE * 2 * NP; k += BS) {
    const int r = k % NP, d = (k / NP) & 1, en = k / (2 * NP), x = en % TX, y = en / TX;
    if (x < tw && y < th) {
      const int f0 = d ? NX + y * TX + x : y * (TX + 1) + x, f1 = f0 + (d ? TX : 1);
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NU; ++q)
        s = fmax(s, su[(q * (NX + NY) + f0) * NP + r] + su[(q * (NX + NY) + f1) * NP + r]);
      const double a = samp[d][d ? x : y];
      ssg[en][d * NP + r] = a > 0.0 ? H->fr[r] * s / a : 0.0;
    }
  }
  __syncthreads();
  for (int k = tid; k < TE * NP; k += BS) {
    const int l = k % NP, en = k / NP, x = en % TX, y = en / TX;
    if (x < tw && y < th) {
      double ax = 0.0, ay = 0.0, sgx = 0.0, sgy = 0.0;
#pragma unroll
      for (int j = 0; j < NP; ++j) { ax = fmax(ax, sws[0][j][en]); ay = fmax(ay, sws[1][j][en]); }
      const double lx = (2.0 * P + 1.0) * mp.rhx * ax, ly = (2.0 * P + 1.0) * mp.rhy * ay;
      for (int r = 0; r <= l; ++r) { sgx += ssg[en][r]; sgy += ssg[en][NP + r]; }
      Dfac[(long)((ty0 + y) * mp.nx + tx0 + x) * NP + l] = l == 0 ? 1.0 : exp(-sM * tau * (lx * sgx + ly * sgy));
    }
  }
}

template <int P, int M, bool R2, int S>
__global__ __launch_bounds__((VS<P, M, R2, S>::BS)) void k_vel_sensor(const double* __restrict__ rho, const double* __restrict__ u,
                                                    const double* __restrict__ Bx, const double* __restrict__ By,
                                                    const double* __restrict__ Bz, const double* __restrict__ lines,
                                                    const double* __restrict__ glob, double* __restrict__ Dfac,
                                                    const HydroTab* __restrict__ H, const MagTab* __restrict__ T,
                                                    MeshP mp, double tau, double sM) {
  vel_sensor_body<P, M, R2, S>(rho, u, Bx, By, Bz, lines, glob, Dfac, H, T, mp, tau, sM, (int)xcd_block());
}

struct vel_sensor_args {
  const double* rho;
  const double* u;
  const double* Bx;
  const double* By;
  const double* Bz;
  const double* lines;
  const double* glob;
  double* Dfac;
  const HydroTab* H;
  const MagTab* T;
  MeshP mp;
  double tau;
  double sM;
};

template <int P, int M, bool R2, int S>
__global__ __launch_bounds__((VS<P, M, R2, S>::BS)) void k_vel_sensor_rt(const vel_sensor_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const vel_sensor_args& a = A[r];
  vel_sensor_body<P, M, R2, S>(gl(a.rho), gl(a.u), gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.lines), gl(a.glob), gl(a.Dfac), gl(a.H), gl(a.T), a.mp, a.tau, a.sM, (int)blockIdx.x - boff[r]);
}

// Velocity-OE map (eq. magnetic-oe-map) with the prepared basis, EB elements per block.  The block's
// basis tables (the p^2 modes of the shells 0..p-1) are copied to LDS first (all of a thread's 16-byte
// loads are issued before the first store; rows keep an odd LDS stride), so the basis is read from
// HBM once (5.5 GB, 4.6 of them read, at 1024^2, N = 4 in 0.995 ms: 5.5 TB/s).  Then the coefficients
// c_k = (u_d, psi_k)_rho (task = element and mode) and the shells' parts at the nodes (thread = node) are
// formed, the last shell's part as what the others leave of u, and u and e are updated in place.
template <int P, int BS>
struct VPJ {
  static constexpr int NP = P + 1, NN = NP * NP, NK = psi_modes(P), EB = BS / NN, NKP = NK | 1;
  static constexpr long PS = psi_stride(P), RS = psi_row(P);
};

template <int P, int BS, bool R2>
__device__ __forceinline__ void vel_proj_body(const double* __restrict__ rho, double* __restrict__ u,
                                                  double* __restrict__ en, const double* __restrict__ Psi,
                                                  const double* __restrict__ Dfac, const HydroTab* __restrict__ H,
                                                  MeshP mp, double* __restrict__ Uc, long blk) {
  using C = VPJ<P, BS>;
  constexpr int NP = C::NP, NN = C::NN, NK = C::NK, EB = C::EB, NKP = C::NKP, NU = R2 ? 2 : 3;
  constexpr int PS = (int)C::PS, RS = (int)C::RS;
  __shared__ double sP[EB * NN * NKP];
  __shared__ double sv[EB][NU][NN], sc[EB][NU][NK], sD[EB][NP];
  const int tid = threadIdx.x, el = tid / NN, q = tid - el * NN;
  const int qi = q % NP, qj = q / NP;
  const long e0 = blk * EB, e = e0 + el;
  const int nel = mp.K - e0 < EB ? (int)(mp.K - e0) : EB;
  const bool act = el < nel;
  const long KN = mp.K * NN;
  {
    constexpr int NL = (EB * PS / 2 + BS - 1) / BS;
    const int n2 = nel * PS / 2;
    const double2* src = reinterpret_cast<const double2*>(Psi + e0 * PS);
    double2 v[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int t = tid + BS * k;
      v[k] = t < n2 ? src[t] : double2{0.0, 0.0};
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int t = tid + BS * k;
      if (t < n2) {
        // RS even: both values lie in one row (element and node), columns c0 and c0 + 1 (padding skipped)
        const int r = 2 * t / RS, c0 = 2 * t - r * RS;
        double* d = sP + r * NKP + c0;
        d[0] = v[k].x;
        if (NK % 2 == 0 || c0 + 1 < NK) d[1] = v[k].y;
      }
    }
  }
  double rq = 0.0, uo[3] = {0.0, 0.0, 0.0};
  if (act) {
    rq = rho[e * NN + q];
    const double wq = mp.J * H->w[qi] * H->w[qj] * rq;
#pragma unroll
    for (int d = 0; d < NU; ++d) {  // u_z = 0 in 2D2V
      uo[d] = u[d * KN + e * NN + q];
      sv[el][d][q] = wq * uo[d];
    }
    if (q < NP) sD[el][q] = Dfac[e * NP + q];
  }
  __syncthreads();
  for (int t = tid; t < nel * NK; t += BS) {
    const int ee = t / NK, k = t - ee * NK;
    const double* Pe = sP + ee * NN * NKP + k;  // Pe[n * NKP] = psi_k(x_n)
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int n = 0; n < NN; ++n) {
      const double pn = Pe[n * NKP];
#pragma unroll
      for (int d = 0; d < NU; ++d) s[d] += sv[ee][d][n] * pn;
    }
#pragma unroll
    for (int d = 0; d < NU; ++d) sc[ee][d][k] = s[d];
  }
  __syncthreads();
  if (!act) return;
  double wl[3][NP];
#pragma unroll
  for (int d = 0; d < NU; ++d)
#pragma unroll
    for (int l = 0; l < P; ++l) wl[d][l] = 0.0;
  const double* Pq = sP + tid * NKP;
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const double pk = Pq[k];
#pragma unroll
    for (int d = 0; d < NU; ++d) wl[d][shell_of(k)] += sc[el][d][k] * pk;
  }
  double heat = 0.0, un[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int d = 0; d < NU; ++d) {
    double v = wl[d][0], rest = uo[d] - v;
#pragma unroll
    for (int l = 1; l < P; ++l) rest -= wl[d][l];
    wl[d][P] = rest;
#pragma unroll
    for (int l = 1; l < NP; ++l) {
      const double Dl = sD[el][l];
      v += Dl * wl[d][l];
      heat += 0.5 * (1.0 - Dl * Dl) * wl[d][l] * wl[d][l];
    }
    un[d] = v;
  }
  const long n = e * NN + q;
  if (!Uc) {
#pragma unroll
    for (int d = 0; d < NU; ++d) u[d * KN + n] = un[d];
    en[n] += heat;
  } else {
    // last stage of a Strang step's magnetic substep: the exchange back to the conserved state
    // (section "Local variable exchange") is formed here instead of by a separate pass; the density
    // row of Uc already holds rho, and the primitive copies are not needed afterwards
    const double ev = en[n] + heat;
    Uc[KN + n] = rq * un[0]; Uc[2 * KN + n] = rq * un[1]; Uc[3 * KN + n] = rq * un[2];
    Uc[4 * KN + n] = rq * ev + 0.5 * rq * (un[0] * un[0] + un[1] * un[1] + un[2] * un[2]);
  }
}

template <int P, int BS, bool R2>
__global__ __launch_bounds__(BS) void k_vel_proj(const double* __restrict__ rho, double* __restrict__ u,
                                                  double* __restrict__ en, const double* __restrict__ Psi,
                                                  const double* __restrict__ Dfac, const HydroTab* __restrict__ H,
                                                  MeshP mp, double* __restrict__ Uc) {
  vel_proj_body<P, BS, R2>(rho, u, en, Psi, Dfac, H, mp, Uc, (long)blockIdx.x);
}

struct vel_proj_args {
  const double* rho;
  double* u;
  double* en;
  const double* Psi;
  const double* Dfac;
  const HydroTab* H;
  MeshP mp;
  double* Uc;
};

template <int P, int BS, bool R2>
__global__ __launch_bounds__(BS) void k_vel_proj_rt(const vel_proj_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const vel_proj_args& a = A[r];
  vel_proj_body<P, BS, R2>(gl(a.rho), gl(a.u), gl(a.en), gl(a.Psi), gl(a.Dfac), gl(a.H), a.mp, gl(a.Uc), (long)blockIdx.x - boff[r]);
}

// ---------------------------------------------------------------------------------------------
// Artificial resistivity (eq. magnetic-ar-sensor, eq. magnetic-ar-coefficient) in two passes.
// Pass 1 (one thread per GLL_p node, B coefficients staged in LDS): each element's tangential
// traces on its four faces at the (m+2) face Gauss points and the element maxima of |u_I| + |B|/sqrt(rho)
// over its GLL_p nodes -> tr[K][8A + 2], trace index ((dir*2 + it)*2 + side)*A + k; dir 0 holds the
// x-faces (it 0: B_y, it 1: B_z), dir 1 the y-faces (it 0: B_x, it 1: B_z); side 0 is the face at -1.
// Pass 2 (one thread per element): squared jumps against the neighbours' traces, sigma^B, R, eta.
// ---------------------------------------------------------------------------------------------
template <int P, int M>
__device__ __forceinline__ void ar_traces_body(const double* __restrict__ rho, const double* __restrict__ u,
                                                   const double* __restrict__ Bx, const double* __restrict__ By,
                                                   const double* __restrict__ Bz, double* __restrict__ tr,
                                                   const MagTab* __restrict__ T, MeshP mp, long blk) {
  constexpr int NP = P + 1, NN = NP * NP, EB = 256 / NN, A = M + 2, B = M + 1, AB = A * B, BB = B * B;
  constexpr int NT = 8 * A + 2;
  __shared__ double sbx[EB][AB], sby[EB][AB], sbz[EB][BB], sv[EB][2][NN];
  __shared__ double tWP[NP][A], tGP[NP][B], tVP[NP][B], tWQ[A][A], tVQ[A][B], tGE[2][B], tVE[2][B];
  const int tid = threadIdx.x, el = tid / NN, q = tid - el * NN, qi = q % NP, qj = q / NP;
  const long e = blk * EB + el;
  const bool act = el < EB && e < mp.K;
  long ex, ey;
  elem_xy(mp, act ? e : 0, ex, ey);
  const long KN = mp.K * NN;
  for (int t = tid; t < NP * A; t += 256) tWP[t / A][t % A] = T->I_W_P[t / A][t % A];
  for (int t = tid; t < NP * B; t += 256) {
    tGP[t / B][t % B] = T->I_G_P[t / B][t % B];
    tVP[t / B][t % B] = T->I_V_P[t / B][t % B];
  }
  for (int t = tid; t < A * A; t += 256) tWQ[t / A][t % A] = T->I_W_Q[t / A][t % A];
  for (int t = tid; t < A * B; t += 256) tVQ[t / B][t % B] = T->I_V_Q[t / B][t % B];
  for (int t = tid; t < 2 * B; t += 256) {
    tGE[t / B][t % B] = T->I_G_E[t / B][t % B];
    tVE[t / B][t % B] = T->I_V_E[t / B][t % B];
  }
  if (act) {
    for (int k = q; k < AB; k += NN) {
      sbx[el][k] = Bx[gix(mp, B, ex, ey, k % A, k / A)];  // [j<B][i<A]
      sby[el][k] = By[gix(mp, B, ex, ey, k % B, k / B)];  // [j<A][i<B]
    }
    for (int k = q; k < BB; k += NN) sbz[el][k] = Bz[gix(mp, B, ex, ey, k % B, k / B)];
  }
  __syncthreads();
  double* o = tr + (act ? e : 0) * NT;
  if (act) {
    double bxv = 0.0, byv = 0.0, bzv = 0.0;
    // the outer loops stay rolled: unrolled, the scheduler hoists every LDS operand of the three
    // evaluations at once (170 VGPRs, 2 waves per SIMD)
#pragma unroll 1
    for (int j = 0; j < B; ++j) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < A; ++i) s += tWP[qi][i] * sbx[el][j * A + i];
      bxv += tGP[qj][j] * s;
    }
#pragma unroll 1
    for (int j = 0; j < A; ++j) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < B; ++i) s += tGP[qi][i] * sby[el][j * B + i];
      byv += tWP[qj][j] * s;
    }
#pragma unroll 1
    for (int j = 0; j < B; ++j) {
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < B; ++i) s += tVP[qi][i] * sbz[el][j * B + i];
      bzv += tVP[qj][j] * s;
    }
    const double va = sqrt(bxv * bxv + byv * byv + bzv * bzv) * rsqrt_refined(rho[e * NN + q]);  // rho > 0
    sv[el][0][q] = fabs(u[e * NN + q]) + va;
    sv[el][1][q] = fabs(u[KN + e * NN + q]) + va;
    for (int t = q; t < 8 * A; t += NN) {
      const int k = t % A, s = (t / A) % 2, it = (t / (2 * A)) % 2, dir = t / (4 * A);
      double v = 0.0;
      if (it == 1) {  // B_z: GLL_m x GLL_m
        for (int j = 0; j < B; ++j)
          for (int i = 0; i < B; ++i)
            v += (dir == 0 ? tVE[s][i] * tVQ[k][j] : tVQ[k][i] * tVE[s][j]) * sbz[el][j * B + i];
      } else if (dir == 0) {  // B_y on x-faces: Gauss_m in x, GLL_{m+1} in y
        for (int j = 0; j < A; ++j)
          for (int i = 0; i < B; ++i) v += tGE[s][i] * tWQ[k][j] * sby[el][j * B + i];
      } else {  // B_x on y-faces: GLL_{m+1} in x, Gauss_m in y
        for (int j = 0; j < B; ++j)
          for (int i = 0; i < A; ++i) v += tWQ[k][i] * tGE[s][j] * sbx[el][j * A + i];
      }
      o[t] = v;
    }
  }
  __syncthreads();
  if (act && q < 2) {
    double m = 0.0;
    for (int k = 0; k < NN; ++k) m = fmax(m, sv[el][q][k]);
    o[8 * A + q] = m;
  }
}

template <int P, int M>
__global__ __launch_bounds__(256) void k_ar_traces(const double* __restrict__ rho, const double* __restrict__ u,
                                                   const double* __restrict__ Bx, const double* __restrict__ By,
                                                   const double* __restrict__ Bz, double* __restrict__ tr,
                                                   const MagTab* __restrict__ T, MeshP mp) {
  ar_traces_body<P, M>(rho, u, Bx, By, Bz, tr, T, mp, (long)blockIdx.x);
}

struct ar_traces_args {
  const double* rho;
  const double* u;
  const double* Bx;
  const double* By;
  const double* Bz;
  double* tr;
  const MagTab* T;
  MeshP mp;
};

template <int P, int M>
__global__ __launch_bounds__(256) void k_ar_traces_rt(const ar_traces_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const ar_traces_args& a = A[r];
  ar_traces_body<P, M>(gl(a.rho), gl(a.u), gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.tr), gl(a.T), a.mp, (long)blockIdx.x - boff[r]);
}

// bglob[3][3]: (integral, min, max) of B_x, B_y, B_z over the domain.
template <int P, int M>
__device__ __forceinline__ void ar_eta_body(const double* __restrict__ tr, const double* __restrict__ bglob,
                                                double* __restrict__ eta, const MagTab* __restrict__ T, MeshP mp,
                                                double Cs, double Ceta, long blk) {
  constexpr int A = M + 2, NT = 8 * A + 2;
  const long e = blk * blockDim.x + threadIdx.x;
  if (e >= mp.K) return;
  long ex, ey;
  elem_xy(mp, e, ex, ey);
  double dOm[3];
  bool cf[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double mean = bglob[c * 3] / mp.area, mn = bglob[c * 3 + 1], mx = bglob[c * 3 + 2];
    dOm[c] = fmax(mx - mean, mean - mn);
    cf[c] = mx - mn <= 1024.0 * EPSM * fmax(fabs(mx), fabs(mn));  // roundoff-level variation (exact test)
  }
  const double* me = tr + e * NT;
  double R[2];
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    const int t0 = dir == 0 ? 1 : 0;
    const double DB = fmax(cf[t0] ? 0.0 : dOm[t0], cf[2] ? 0.0 : dOm[2]);
    double sig = 0.0;
    if (DB > 0.0) {
      const long em = dir == 0 ? ey * mp.nx + wrapl(ex - 1, mp.nx) : wrapl(ey - 1, mp.ny) * mp.nx + ex;
      const long ep = dir == 0 ? ey * mp.nx + wrapl(ex + 1, mp.nx) : wrapl(ey + 1, mp.ny) * mp.nx + ex;
      const double* tm = tr + em * NT;
      const double* tp = tr + ep * NT;
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        if (cf[it == 0 ? t0 : 2]) continue;
        const int b0 = (dir * 2 + it) * 2 * A, b1 = b0 + A;  // side 0 / side 1 blocks
        double sm = 0.0, sp = 0.0;
        for (int k = 0; k < A; ++k) {
          const double jm = me[b0 + k] - tm[b1 + k];
          const double jp = tp[b0 + k] - me[b1 + k];
          sm += 0.5 * T->wq[k] * jm * jm;
          sp += 0.5 * T->wq[k] * jp * jp;
        }
        sig = fmax(sig, (sqrt(sm) + sqrt(sp)) / (2.0 * DB));
      }
    }
    R[dir] = fmin(Cs * sig, 1.0);
  }
  const double v0 = mp.hx / (2.0 * P + 1.0) * me[8 * A] * R[0];
  const double v1 = mp.hy / (2.0 * P + 1.0) * me[8 * A + 1] * R[1];
  eta[e] = Ceta * fmax(v0, v1);
}

template <int P, int M>
__global__ __launch_bounds__(256) void k_ar_eta(const double* __restrict__ tr, const double* __restrict__ bglob,
                                                double* __restrict__ eta, const MagTab* __restrict__ T, MeshP mp,
                                                double Cs, double Ceta) {
  ar_eta_body<P, M>(tr, bglob, eta, T, mp, Cs, Ceta, (long)blockIdx.x);
}

struct ar_eta_args {
  const double* tr;
  const double* bglob;
  double* eta;
  const MagTab* T;
  MeshP mp;
  double Cs;
  double Ceta;
};

template <int P, int M>
__global__ __launch_bounds__(256) void k_ar_eta_rt(const ar_eta_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const ar_eta_args& a = A[r];
  ar_eta_body<P, M>(gl(a.tr), gl(a.bglob), gl(a.eta), gl(a.T), a.mp, a.Cs, a.Ceta, (long)blockIdx.x - boff[r]);
}

// per-element exact integral and owned-node min / max of each B component -> [K][3][3]
template <int M>
__device__ __forceinline__ void B_stats_body(const double* __restrict__ Bx, const double* __restrict__ By,
                                                 const double* __restrict__ Bz, double* __restrict__ stats,
                                                 const MagTab* __restrict__ T, MeshP mp, long blk) {
  constexpr int A = M + 2, B = M + 1;
  const long e = blk * blockDim.x + threadIdx.x;
  if (e >= mp.K) return;
  long ex, ey;
  elem_xy(mp, e, ex, ey);
  double s[3] = {0, 0, 0}, mn[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, mx[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
  // extrema over the element's own DOFs (its upper shared nodes belong to the next element); on a
  // mirror-walled mesh the box's last column / row of elements also takes the box's wall DOFs
  const bool wx = (mp.walls & 1) && ex == mp.bx - 1, wy = (mp.walls & 2) && ey == mp.by - 1;
  // outer loops rolled: fully unrolled, the three loops keep every load in flight at once (about
  // 190 VGPRs, 2 waves per SIMD instead of 6)
#pragma unroll 1
  for (int j = 0; j < B; ++j)
    for (int i = 0; i < A; ++i) {
      const double v = Bx[gix(mp, B, ex, ey, i, j)];
      s[0] += T->ww[i] * T->wg[j] * v;
      if (i < B || wx) { mn[0] = fmin(mn[0], v); mx[0] = fmax(mx[0], v); }
    }
#pragma unroll 1
  for (int j = 0; j < A; ++j)
    for (int i = 0; i < B; ++i) {
      const double v = By[gix(mp, B, ex, ey, i, j)];
      s[1] += T->wg[i] * T->ww[j] * v;
      if (j < B || wy) { mn[1] = fmin(mn[1], v); mx[1] = fmax(mx[1], v); }
    }
#pragma unroll 1
  for (int j = 0; j < B; ++j)
    for (int i = 0; i < B; ++i) {
      const double v = Bz[gix(mp, B, ex, ey, i, j)];
      s[2] += T->wv[i] * T->wv[j] * v;
      mn[2] = fmin(mn[2], v); mx[2] = fmax(mx[2], v);
    }
  for (int c = 0; c < 3; ++c) {
    stats[(e * 3 + c) * 3] = mp.J * s[c];
    stats[(e * 3 + c) * 3 + 1] = mn[c];
    stats[(e * 3 + c) * 3 + 2] = mx[c];
  }
}

template <int M>
__global__ __launch_bounds__(256) void k_B_stats(const double* __restrict__ Bx, const double* __restrict__ By,
                                                 const double* __restrict__ Bz, double* __restrict__ stats,
                                                 const MagTab* __restrict__ T, MeshP mp) {
  B_stats_body<M>(Bx, By, Bz, stats, T, mp, (long)blockIdx.x);
}

struct B_stats_args {
  const double* Bx;
  const double* By;
  const double* Bz;
  double* stats;
  const MagTab* T;
  MeshP mp;
};

template <int M>
__global__ __launch_bounds__(256) void k_B_stats_rt(const B_stats_args* __restrict__ A, const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const B_stats_args& a = A[r];
  B_stats_body<M>(gl(a.Bx), gl(a.By), gl(a.Bz), gl(a.stats), gl(a.T), a.mp, (long)blockIdx.x - boff[r]);
}

}  // namespace

// Local-to-global maps of the six magnetic node sets of each element (B_x, B_y, B_z, W, N_x, N_y;
// local order [j][i], i fastest), formed with the kernels' own grid index gix.  One thread per element.
template <int M>
__global__ __launch_bounds__(256) void k_dof_maps(int32_t* __restrict__ dof, MeshP mp) {
  constexpr int A = M + 2, B = M + 1;
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= mp.K) return;
  long ex, ey;
  elem_xy(mp, e, ex, ey);
  const int ni[6] = {A, B, B, A, B, A}, nj[6] = {B, A, B, A, A, B};
  long off = 0;
  for (int s = 0; s < 6; ++s) {
    const int n = ni[s] * nj[s];
    int32_t* o = dof + off + e * n;
    for (int j = 0; j < nj[s]; ++j)
      for (int i = 0; i < ni[s]; ++i) o[j * ni[s] + i] = (int32_t)gix(mp, B, ex, ey, i, j);
    off += mp.K * n;
  }
}

// Admissibility test of a magnetic-substep input: rho > 0, e > 0 (p = (gamma - 1) rho e > 0) and
// finite u at every node, finite magnetic grids.  A failure sets bit 1 of flag[1].
__global__ __launch_bounds__(256) void k_check_mag(const double* __restrict__ rho, const double* __restrict__ e,
                                                   const double* __restrict__ u, long KN, const double* __restrict__ Bx,
                                                   const double* __restrict__ By, const double* __restrict__ Bz, long G,
                                                   int* __restrict__ flag) {
  const long n = KN > G ? KN : G;
  bool ok = true;
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x) {
    if (k < KN) {
      const double r = rho[k], en = e[k];
      ok = ok && r > 0.0 && en > 0.0 && r <= DBL_MAX && en <= DBL_MAX && fabs(u[k]) <= DBL_MAX &&
           fabs(u[KN + k]) <= DBL_MAX && fabs(u[2 * KN + k]) <= DBL_MAX;
    }
    if (k < G) ok = ok && fabs(Bx[k]) <= DBL_MAX && fabs(By[k]) <= DBL_MAX && fabs(Bz[k]) <= DBL_MAX;
  }
  if (!ok) atomicOr(flag + 1, 2);
}

__device__ __forceinline__ void to_primitive_node(const double* __restrict__ U, double* __restrict__ rho,
                                                  double* __restrict__ e, double* __restrict__ u, long n, long k) {
  const double r = U[k], ux = U[n + k] / r, uy = U[2 * n + k] / r, uz = U[3 * n + k] / r;
  rho[k] = r; u[k] = ux; u[n + k] = uy; u[2 * n + k] = uz;
  e[k] = internal_energy(U[4 * n + k], r, ux, uy, uz);
}

__device__ __forceinline__ void to_conservative_node(const double* __restrict__ rho, const double* __restrict__ e,
                                                     const double* __restrict__ u, double* __restrict__ U, long n,
                                                     long k) {
  const double r = rho[k], ux = u[k], uy = u[n + k], uz = u[2 * n + k];
  U[k] = r; U[n + k] = r * ux; U[2 * n + k] = r * uy; U[3 * n + k] = r * uz;
  U[4 * n + k] = r * e[k] + 0.5 * r * (ux * ux + uy * uy + uz * uz);
}

__global__ void k_to_primitive(const double* __restrict__ U, double* __restrict__ rho, double* __restrict__ e,
                               double* __restrict__ u, long n) {
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x)
    to_primitive_node(U, rho, e, u, n, k);
}

__global__ void k_to_conservative(const double* __restrict__ rho, const double* __restrict__ e,
                                  const double* __restrict__ u, double* __restrict__ U, long n) {
  for (long k = (long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long)gridDim.x * blockDim.x)
    to_conservative_node(rho, e, u, U, n, k);
}

// B_par = (-d_y A, d_x A) for A on the E_z grid
template <int M>
__global__ void k_B_from_potential(const double* __restrict__ Az, double* __restrict__ Bx, double* __restrict__ By,
                                   const MagTab* __restrict__ T, MeshP mp) {
  constexpr int A = M + 2, B = M + 1;
  const long NX = (long)mp.nx * B, G = NX * mp.ny * B;
  const long g = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= G) return;
  const long gy = row_of(mp, g / B), gx = g - gy * NX;  // g / (nx B) = (g / B) / nx
  const long ex = gx / B, ey = gy / B;
  const int i = gx - ex * B, j = gy - ey * B;
  double bx = 0.0, by = 0.0;
  for (int k = 0; k < A; ++k) {
    bx += T->D_W_G[j][k] * Az[gix(mp, B, ex, ey, i, k)];  // B_x node: GLL i, Gauss j
    by += T->D_W_G[i][k] * Az[gix(mp, B, ex, ey, k, j)];  // B_y node: Gauss i, GLL j
  }
  Bx[g] = -(2.0 / mp.hy) * bx;
  By[g] = (2.0 / mp.hx) * by;
}

// ---------------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------------
int line_global_reduce(mhd25_ctx* c, const double* stats, int nc, const int* flag);
int dcopy(mhd25_ctx* c, const double* a, double* b, long n);

static int chk(mhd25_ctx* c, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { c->err = std::string(what) + ": " + hipGetErrorString(e); return -2; }
  return 0;
}

hipEvent_t* timing_slot(mhd25_ctx* c, int kid, int inner = 0);
// HIP-event timing of one launch (kernel id kid) when the context's timing is on
#define T_BEGIN(kid)                                                   \
  hipEvent_t* ev_ = c->timing ? timing_slot(c, kid) : nullptr;         \
  if (ev_) hipEventRecord(ev_[0], c->stream)
#define T_END() \
  if (ev_) hipEventRecord(ev_[1], c->stream)

#define DISPATCH_PM(p, m, F)                                                                              \
  if (p == 1 && m == 0) { F(1, 0); } else if (p == 1 && m == 1) { F(1, 1); }                              \
  else if (p == 2 && m == 1) { F(2, 1); } else if (p == 2 && m == 2) { F(2, 2); }                         \
  else if (p == 3 && m == 2) { F(3, 2); } else if (p == 3 && m == 3) { F(3, 3); }                         \
  else if (p == 4 && m == 3) { F(4, 3); } else if (p == 4 && m == 4) { F(4, 4); }                         \
  else if (p == 5 && m == 4) { F(5, 4); } else if (p == 5 && m == 5) { F(5, 5); }                         \
  else if (p == 6 && m == 5) { F(6, 5); } else if (p == 6 && m == 6) { F(6, 6); }                         \
  else return -4;

#define DISPATCH_M(m, F) \
  switch (m) { case 0: F(0); break; case 1: F(1); break; case 2: F(2); break; case 3: F(3); break; \
               case 4: F(4); break; case 5: F(5); break; case 6: F(6); break; default: return -4; }

// template keys of run-table records: degree p, magnetic degree m, 2D2V flag, mode
static int mkey(int p, int m, bool r2, int mode = 0) { return p * 1000 + m * 100 + (r2 ? 10 : 0) + mode; }

static long mblocks(int p, int m, long K, int bs = 256) {
  const int nn = (p + 1) * (p + 1), aa = (m + 2) * (m + 2);
  const int eb = bs / (nn > aa ? nn : aa);
  return (K + eb - 1) / eb;
}

// threads per block of the update kernel
#ifndef MHD_MU_BS
#define MHD_MU_BS 256
#endif
// threads per block of the velocity-OE projection (its per-element basis tile in LDS sets how
// many blocks share a CU)
#ifndef MHD_VP_BS
#define MHD_VP_BS 128
#endif

// tile shape of the tile kernels (see RT)
static int mesh_shape(const MeshP& mp) { return mp.ny == 1 && mp.nx > 1 ? 1 : (mp.nx == 1 && mp.ny > 1 ? 2 : 0); }
template <class C>
static dim3 tiles(const MeshP& mp) {
  return dim3((unsigned)((long)((mp.nx + C::TX - 1) / C::TX) * ((mp.ny + C::TY - 1) / C::TY)));
}
// F(R2, S) for the context's system and shape
#define DISPATCH_RS(r2, sh, F)                                                                            \
  if (sh == 0) { if (r2) { F(true, 0); } else { F(false, 0); } }                                          \
  else if (sh == 1) { if (r2) { F(true, 1); } else { F(false, 1); } }                                     \
  else { if (r2) { F(true, 2); } else { F(false, 2); } }

template <int M>
static long recon_tiles(const mhd25_ctx* c, int sh) {
  long nb = 0;
#define NB(R2, S) nb = tiles<RT<M, R2, S>>(c->mp).x
  DISPATCH_RS(false, sh, NB);
#undef NB
  return nb;
}
template <int M>
static void launch_J(mhd25_ctx* c, const J_args& a, bool r2, int sh) {
#define GO(R2, S) hipLaunchKernelGGL((k_J<M, R2, S>), (tiles<RT<M, R2, S>>(c->mp)), dim3(RT<M, R2, S>::BS), 0, c->stream, \
                                     a.Bx, a.By, a.Bz, a.Jx, a.Jy, a.Jz, a.T, a.mp)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}
template <int P, int M>
static void launch_E(mhd25_ctx* c, const E_args& a, bool r2, int sh) {
#define GO(R2, S) hipLaunchKernelGGL((k_E<P, M, R2, S>), (tiles<RT<M, R2, S>>(c->mp)), dim3(RT<M, R2, S>::BS), 0, c->stream, \
                                     a.u, a.Bx, a.By, a.Bz, a.Jx, a.Jy, a.Jz, a.eta, a.Ex, a.Ey, a.Ez, a.T, a.mp)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}

// J alone (three grids).  r2: the 2D2V reduced system (only J_z and E_z are formed; the in-plane grids are not written)
int mag_reconstruct_J(mhd25_ctx* c, const double* Bx, const double* By, const double* Bz, double* J, bool r2) {
  const J_args a{Bx, By, Bz, J, J + c->G, J + 2 * c->G, c->d_mt, c->mp};
  const int sh = mesh_shape(c->mp);
  if (c->rec) {
    long nb = 0;
#define NB(M) nb = recon_tiles<M>(c, sh)
    DISPATCH_M(c->m, NB);
#undef NB
    rt_record(c, RT_J, mkey(c->p, c->m, r2, sh), nb, a);
    return 0;
  }
#define LJ(M) launch_J<M>(c, a, r2, sh)
  {
    T_BEGIN(7);
    DISPATCH_M(c->m, LJ);
    T_END();
  }
#undef LJ
  return chk(c, "J reconstruction launch");
}

int mag_reconstruct_JE(mhd25_ctx* c, const double* u, const double* Bx, const double* By, const double* Bz,
                       const double* eta, double* JE, bool r2) {
  const long G = c->G;
  if (const int r = mag_reconstruct_J(c, Bx, By, Bz, JE, r2)) return r;
  const E_args a{u, Bx, By, Bz, JE, JE + G, JE + 2 * G, eta, JE + 3 * G, JE + 4 * G, JE + 5 * G, c->d_mt, c->mp};
  const int sh = mesh_shape(c->mp);
  if (c->rec) {
    long nb = 0;
#define NB(M) nb = recon_tiles<M>(c, sh)
    DISPATCH_M(c->m, NB);
#undef NB
    rt_record(c, RT_E, mkey(c->p, c->m, r2, sh), nb, a);
    return 0;
  }
#define LE(P, M) (launch_E<P, M>(c, a, r2, sh))
  {
    T_BEGIN(5);
    DISPATCH_PM(c->p, c->m, LE);
    T_END();
  }
#undef LE
  return chk(c, "reconstruct launch");
}

template <int P, int M>
static long sensor_tiles(const mhd25_ctx* c, bool r2, int sh) {
  long nb = 0;
#define NB(R2, S) nb = tiles<VS<P, M, R2, S>>(c->mp).x
  DISPATCH_RS(r2, sh, NB);
#undef NB
  return nb;
}
template <int P, int M>
static void launch_vel_sensor(mhd25_ctx* c, const vel_sensor_args& a, bool r2, int sh) {
#define GO(R2, S) hipLaunchKernelGGL((k_vel_sensor<P, M, R2, S>), (tiles<VS<P, M, R2, S>>(c->mp)), dim3((VS<P, M, R2, S>::BS)), 0, \
                                     c->stream, a.rho, a.u, a.Bx, a.By, a.Bz, a.lines, a.glob, a.Dfac, a.H, a.T, a.mp, a.tau, a.sM)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}

int mag_update(mhd25_ctx* c, const MagIO& io, int mode) {
  const long nb = mblocks(c->p, c->m, c->mp.K, MHD_MU_BS);
  const bool r2 = c->opt.reduced_2d2v != 0;
  if (c->rec) { rt_record(c, RT_MAG_UPDATE, mkey(c->p, c->m, r2, mode), nb, mag_update_args{io, c->d_mt, c->mp}); return 0; }
#define U0(P, M)                                                                                                    \
  if (r2) hipLaunchKernelGGL((k_mag_update<P, M, 0, MHD_MU_BS, true>), dim3(nb), dim3(MHD_MU_BS), 0, c->stream, io, \
                             c->d_mt, c->mp);                                                                        \
  else hipLaunchKernelGGL((k_mag_update<P, M, 0, MHD_MU_BS, false>), dim3(nb), dim3(MHD_MU_BS), 0, c->stream, io,   \
                          c->d_mt, c->mp)
#define U1(P, M)                                                                                                    \
  if (r2) hipLaunchKernelGGL((k_mag_update<P, M, 1, MHD_MU_BS, true>), dim3(nb), dim3(MHD_MU_BS), 0, c->stream, io, \
                             c->d_mt, c->mp);                                                                        \
  else hipLaunchKernelGGL((k_mag_update<P, M, 1, MHD_MU_BS, false>), dim3(nb), dim3(MHD_MU_BS), 0, c->stream, io,   \
                          c->d_mt, c->mp)
  T_BEGIN(2);
  if (mode == 0) {
    DISPATCH_PM(c->p, c->m, U0);
  } else {
    DISPATCH_PM(c->p, c->m, U1);
  }
  T_END();
#undef U0
#undef U1
  return chk(c, "magnetic update launch");
}

static int vp_eb(int p) {
  switch (p) { case 1: return VP<1>::EB; case 2: return VP<2>::EB; case 3: return VP<3>::EB;
               case 4: return VP<4>::EB; case 5: return VP<5>::EB; default: return VP<6>::EB; }
}

int mag_velocity_prep(mhd25_ctx* c, const double* rho) {
  const long K = c->mp.K;
  const long nn = (long)(c->p + 1) * (c->p + 1);
  (void)nn;
  if (!c->psi) { c->err = "velocity-OE basis not allocated"; return -2; }
  if (c->rec) {
    rt_record(c, RT_VEL_PREP, c->p, (K + vp_eb(c->p) - 1) / vp_eb(c->p),
              vel_prep_args{rho, c->psi, c->d_ht, c->mp});
    return 0;
  }
#define VPR(P) hipLaunchKernelGGL((k_vel_prep<P>), dim3((K + VP<P>::EB - 1) / VP<P>::EB), dim3(MHD_PREP_BS), 0, c->stream, rho, \
                                  c->psi, c->d_ht, c->mp)
  T_BEGIN(4);
  switch (c->p) { case 1: VPR(1); break; case 2: VPR(2); break; case 3: VPR(3); break; case 4: VPR(4); break;
                  case 5: VPR(5); break; case 6: VPR(6); break; default: return -4; }
  T_END();
#undef VPR
  return chk(c, "velocity OE prep launch");
}

int mag_velocity_apply(mhd25_ctx* c, double tau, const double* rho, double* u, double* e, const double* Bx,
                       const double* By, const double* Bz, bool stats_ready, double* Uc) {
  const long K = c->mp.K;
  const int nn = (c->p + 1) * (c->p + 1), eb = 256 / nn, eb2 = MHD_VP_BS / nn;
  const long nb = (K + eb - 1) / eb, nb2 = (K + eb2 - 1) / eb2;
  const bool r2 = c->opt.reduced_2d2v != 0;
  const int nu = r2 ? 2 : 3;  // velocity components carried
  if (!stats_ready && !c->rec) {
#define FS(P)                                                                                                       \
  if (r2) hipLaunchKernelGGL((k_field_stats<P, 2>), dim3(nb), dim3(256), 0, c->stream, u, c->stats, c->d_mt, c->mp); \
  else hipLaunchKernelGGL((k_field_stats<P, 3>), dim3(nb), dim3(256), 0, c->stream, u, c->stats, c->d_mt, c->mp)
    switch (c->p) { case 1: FS(1); break; case 2: FS(2); break; case 3: FS(3); break; case 4: FS(4); break;
                    case 5: FS(5); break; case 6: FS(6); break; default: return -4; }
#undef FS
  }
  line_global_reduce(c, c->stats, nu, nullptr);
  const vel_sensor_args sa{rho, u, Bx, By, Bz, c->lines, c->glob, c->dfac, c->d_ht, c->d_mt, c->mp, tau, c->opt.s_M};
  const int sh = mesh_shape(c->mp);
  if (c->rec) {
    if (!stats_ready) { c->err = "run-table plan: velocity statistics must come from the update"; return -2; }
    long nbs = 0;
#define NBS(P, M) (nbs = sensor_tiles<P, M>(c, r2, sh))
    DISPATCH_PM(c->p, c->m, NBS);
#undef NBS
    rt_record(c, RT_VEL_SENSOR, mkey(c->p, c->m, r2, sh), nbs, sa);
    rt_record(c, RT_VEL_PROJ, mkey(c->p, c->m, r2), nb2, vel_proj_args{rho, u, e, c->psi, c->dfac, c->d_ht, c->mp, Uc});
    return 0;
  }
#define VSN(P, M) (launch_vel_sensor<P, M>(c, sa, r2, sh))
  {
    T_BEGIN(6);
    DISPATCH_PM(c->p, c->m, VSN);
    T_END();
  }
#undef VSN
#define VPR(P)                                                                                                      \
  if (r2) hipLaunchKernelGGL((k_vel_proj<P, MHD_VP_BS, true>), dim3(nb2), dim3(MHD_VP_BS), 0, c->stream, rho, u, e, \
                             c->psi, c->dfac, c->d_ht, c->mp, Uc);                                                    \
  else hipLaunchKernelGGL((k_vel_proj<P, MHD_VP_BS, false>), dim3(nb2), dim3(MHD_VP_BS), 0, c->stream, rho, u, e,   \
                          c->psi, c->dfac, c->d_ht, c->mp, Uc)
  {
    T_BEGIN(3);
    switch (c->p) { case 1: VPR(1); break; case 2: VPR(2); break; case 3: VPR(3); break; case 4: VPR(4); break;
                    case 5: VPR(5); break; case 6: VPR(6); break; default: return -4; }
    T_END();
  }
#undef VPR
  return chk(c, "velocity OE launch");
}

int mag_velocity_oe(mhd25_ctx* c, double tau, const double* rho, double* u, double* e, const double* Bx,
                    const double* By, const double* Bz) {
  int r = mag_velocity_prep(c, rho);
  if (r) return r;
  return mag_velocity_apply(c, tau, rho, u, e, Bx, By, Bz, false, nullptr);
}

int mag_ar_eta(mhd25_ctx* c, const double* rho, const double* u, const double* Bx, const double* By,
               const double* Bz, double* eta) {
  const long K = c->mp.K;
  const long nb = (K + 255) / 256;
  if (c->rec) {
    const long eb = 256 / ((c->p + 1) * (c->p + 1));
    rt_record(c, RT_B_STATS, c->m, nb, B_stats_args{Bx, By, Bz, c->stats, c->d_mt, c->mp});
    line_global_reduce(c, c->stats, 3, nullptr);
    rt_record(c, RT_AR_TRACES, mkey(c->p, c->m, false), (K + eb - 1) / eb,
              ar_traces_args{rho, u, Bx, By, Bz, c->artr, c->d_mt, c->mp});
    rt_record(c, RT_AR_ETA, mkey(c->p, c->m, false), nb,
              ar_eta_args{c->artr, c->glob, eta, c->d_mt, c->mp, c->opt.C_s, c->opt.C_eta});
    return 0;
  }
#define BS(M) hipLaunchKernelGGL((k_B_stats<M>), dim3(nb), dim3(256), 0, c->stream, Bx, By, Bz, c->stats, c->d_mt, c->mp)
  DISPATCH_M(c->m, BS);
#undef BS
  line_global_reduce(c, c->stats, 3, nullptr);
  const long eb = 256 / ((c->p + 1) * (c->p + 1));
  const long nb1 = (K + eb - 1) / eb;
#define ART(P, M) hipLaunchKernelGGL((k_ar_traces<P, M>), dim3(nb1), dim3(256), 0, c->stream, rho, u, Bx, By, Bz, c->artr, \
                                     c->d_mt, c->mp)
  {
    T_BEGIN(9);
    DISPATCH_PM(c->p, c->m, ART);
    T_END();
  }
#undef ART
#define AR(P, M) hipLaunchKernelGGL((k_ar_eta<P, M>), dim3(nb), dim3(256), 0, c->stream, c->artr, c->glob, eta, c->d_mt, \
                                    c->mp, c->opt.C_s, c->opt.C_eta)
  DISPATCH_PM(c->p, c->m, AR);
#undef AR
  return chk(c, "A.R. launch");
}

struct prim_args {
  const double* U;
  double *rho, *e, *u;
  long n;
};

int mag_to_primitive(mhd25_ctx* c, const double* U, double* rho, double* e, double* u) {
  const long n = c->mp.K * c->nn;
  long nb = (n + 255) / 256; if (nb > 65536) nb = 65536;
  if (c->rec) { rt_record(c, RT_TO_PRIM, 0, nb, prim_args{U, rho, e, u, n}); return 0; }
  hipLaunchKernelGGL(k_to_primitive, dim3(nb), dim3(256), 0, c->stream, U, rho, e, u, n);
  return chk(c, "exchange launch");
}

int mag_to_conservative(mhd25_ctx* c, const double* rho, const double* e, const double* u, double* U) {
  const long n = c->mp.K * c->nn;
  long nb = (n + 255) / 256; if (nb > 65536) nb = 65536;
  if (c->rec) { rt_record(c, RT_TO_CONS, 0, nb, prim_args{U, const_cast<double*>(rho), const_cast<double*>(e), const_cast<double*>(u), n}); return 0; }
  hipLaunchKernelGGL(k_to_conservative, dim3(nb), dim3(256), 0, c->stream, rho, e, u, U, n);
  return chk(c, "exchange launch");
}

int entry_clear(mhd25_ctx* c);

int mag_dof_maps(mhd25_ctx* c, int32_t* dof) {
  const long nb = (c->mp.K + 255) / 256;
#define DM(M) hipLaunchKernelGGL((k_dof_maps<M>), dim3(nb), dim3(256), 0, c->stream, dof, c->mp)
  DISPATCH_M(c->m, DM);
#undef DM
  return chk(c, "dof map launch");
}

// clears the entry word flag[1], then tests the magnetic-substep input into it
int mag_check_input(mhd25_ctx* c, const double* rho, const double* e, const double* u, const double* Bx,
                    const double* By, const double* Bz) {
  const long KN = c->mp.K * c->nn, n = KN > c->G ? KN : c->G;
  long nb = (n + 255) / 256; if (nb > 65536) nb = 65536;
  if (const int r = entry_clear(c)) return r;
  hipLaunchKernelGGL(k_check_mag, dim3(nb), dim3(256), 0, c->stream, rho, e, u, KN, Bx, By, Bz, c->G, c->d_flag);
  return chk(c, "input check launch");
}

int mag_B_from_potential(mhd25_ctx* c, const double* A, double* Bx, double* By) {
  const long gb = (c->G + 255) / 256;
#define BP(M) hipLaunchKernelGGL((k_B_from_potential<M>), dim3(gb), dim3(256), 0, c->stream, A, Bx, By, c->d_mt, c->mp)
  DISPATCH_M(c->m, BP);
#undef BP
  return chk(c, "potential launch");
}

// ---------------------------------------------------------------------------------------------
// Run-table launches of this file's kernels (batched ensembles).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_to_primitive_rt(const prim_args* __restrict__ A, const int* __restrict__ boff,
                                                         int nr) {
  const int r = rt_run(boff, nr);
  const prim_args& a = A[r];
  const long stride = (long)(boff[r + 1] - boff[r]) * blockDim.x;
  for (long k = (long)(blockIdx.x - boff[r]) * blockDim.x + threadIdx.x; k < a.n; k += stride)
    to_primitive_node(gl(a.U), gl(a.rho), gl(a.e), gl(a.u), a.n, k);
}

__global__ __launch_bounds__(256) void k_to_conservative_rt(const prim_args* __restrict__ A,
                                                            const int* __restrict__ boff, int nr) {
  const int r = rt_run(boff, nr);
  const prim_args& a = A[r];
  const long stride = (long)(boff[r + 1] - boff[r]) * blockDim.x;
  for (long k = (long)(blockIdx.x - boff[r]) * blockDim.x + threadIdx.x; k < a.n; k += stride)
    to_conservative_node(gl(a.rho), gl(a.e), gl(a.u), const_cast<double*>(gl(a.U)), a.n, k);
}

template <int M>
static void launch_J_rt(bool r2, int sh, dim3 g, hipStream_t s, const J_args* A, const int* dboff, int nr) {
#define GO(R2, S) hipLaunchKernelGGL((k_J_rt<M, R2, S>), g, dim3(RT<M, R2, S>::BS), 0, s, A, dboff, nr)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}
template <int P, int M>
static void launch_E_rt(bool r2, int sh, dim3 g, hipStream_t s, const E_args* A, const int* dboff, int nr) {
#define GO(R2, S) hipLaunchKernelGGL((k_E_rt<P, M, R2, S>), g, dim3(RT<M, R2, S>::BS), 0, s, A, dboff, nr)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}
template <int P, int M>
static void launch_vel_sensor_rt(bool r2, int sh, dim3 g, hipStream_t s, const vel_sensor_args* A, const int* dboff, int nr) {
#define GO(R2, S) hipLaunchKernelGGL((k_vel_sensor_rt<P, M, R2, S>), g, dim3((VS<P, M, R2, S>::BS)), 0, s, A, dboff, nr)
  DISPATCH_RS(r2, sh, GO);
#undef GO
}

int magnetic_rt_launch(const RtRecord& h, const void* dargs, const int* dboff, int nr, long nblocks, hipStream_t s) {
  const dim3 g((unsigned)nblocks);
  const int p = h.key / 1000, m = (h.key / 100) % 10, mode = h.key % 10;
  const bool r2 = (h.key / 10) % 10 != 0;
  switch (h.kind) {
    case RT_J: {
      const J_args* A = (const J_args*)dargs;
#define F(M) launch_J_rt<M>(r2, mode, g, s, A, dboff, nr)
      DISPATCH_M(m, F);
#undef F
      break;
    }
    case RT_E: {
      const E_args* A = (const E_args*)dargs;
#define F(P, M) (launch_E_rt<P, M>(r2, mode, g, s, A, dboff, nr))
      DISPATCH_PM(p, m, F);
#undef F
      break;
    }
    case RT_MAG_UPDATE: {
      const mag_update_args* A = (const mag_update_args*)dargs;
      if (mode != 1) return -2;  // plans hold SSP stages only
#define F(P, M)                                                                                                     \
  if (r2) hipLaunchKernelGGL((k_mag_update_rt<P, M, 1, MHD_MU_BS, true>), g, dim3(MHD_MU_BS), 0, s, A, dboff, nr);  \
  else hipLaunchKernelGGL((k_mag_update_rt<P, M, 1, MHD_MU_BS, false>), g, dim3(MHD_MU_BS), 0, s, A, dboff, nr)
      DISPATCH_PM(p, m, F);
#undef F
      break;
    }
    case RT_VEL_PREP: {
      const vel_prep_args* A = (const vel_prep_args*)dargs;
#define F(P) hipLaunchKernelGGL((k_vel_prep_rt<P>), g, dim3(MHD_PREP_BS), 0, s, A, dboff, nr)
      switch (h.key) { case 1: F(1); break; case 2: F(2); break; case 3: F(3); break; case 4: F(4); break;
                       case 5: F(5); break; case 6: F(6); break; default: return -4; }
#undef F
      break;
    }
    case RT_VEL_SENSOR: {
      const vel_sensor_args* A = (const vel_sensor_args*)dargs;
#define F(P, M) (launch_vel_sensor_rt<P, M>(r2, mode, g, s, A, dboff, nr))
      DISPATCH_PM(p, m, F);
#undef F
      break;
    }
    case RT_VEL_PROJ: {
      const vel_proj_args* A = (const vel_proj_args*)dargs;
#define F(P)                                                                                                        \
  if (r2) hipLaunchKernelGGL((k_vel_proj_rt<P, MHD_VP_BS, true>), g, dim3(MHD_VP_BS), 0, s, A, dboff, nr);          \
  else hipLaunchKernelGGL((k_vel_proj_rt<P, MHD_VP_BS, false>), g, dim3(MHD_VP_BS), 0, s, A, dboff, nr)
      switch (p) { case 1: F(1); break; case 2: F(2); break; case 3: F(3); break; case 4: F(4); break;
                   case 5: F(5); break; case 6: F(6); break; default: return -4; }
#undef F
      break;
    }
    case RT_B_STATS: {
      const B_stats_args* A = (const B_stats_args*)dargs;
#define F(M) hipLaunchKernelGGL((k_B_stats_rt<M>), g, dim3(256), 0, s, A, dboff, nr)
      DISPATCH_M(h.key, F);
#undef F
      break;
    }
    case RT_AR_TRACES: {
      const ar_traces_args* A = (const ar_traces_args*)dargs;
#define F(P, M) hipLaunchKernelGGL((k_ar_traces_rt<P, M>), g, dim3(256), 0, s, A, dboff, nr)
      DISPATCH_PM(p, m, F);
#undef F
      break;
    }
    case RT_AR_ETA: {
      const ar_eta_args* A = (const ar_eta_args*)dargs;
#define F(P, M) hipLaunchKernelGGL((k_ar_eta_rt<P, M>), g, dim3(256), 0, s, A, dboff, nr)
      DISPATCH_PM(p, m, F);
#undef F
      break;
    }
    case RT_TO_PRIM:
      hipLaunchKernelGGL(k_to_primitive_rt, g, dim3(256), 0, s, (const prim_args*)dargs, dboff, nr);
      break;
    case RT_TO_CONS:
      hipLaunchKernelGGL(k_to_conservative_rt, g, dim3(256), 0, s, (const prim_args*)dargs, dboff, nr);
      break;
    default:
      return 1;  // not a kind of this file
  }
  return hipGetLastError() == hipSuccess ? 0 : -2;
}

// ---------------------------------------------------------------------------------------------
// Allocation-free magnetic residual: the same kernels as mhd25_rhs_magnetic, with the
// reconstructed J, E grids in a fixed file-scope device array instead
// of the context's workspace, for callers that cannot allocate device memory.
// ---------------------------------------------------------------------------------------------
namespace {
constexpr long MHD_NOALLOC_DOUBLES = 4L << 20;  // 32 MiB per device
__device__ __align__(256) double scratch[MHD_NOALLOC_DOUBLES];
constexpr int MHD_MAX_DEVICES = 64;
double* g_scratch[MHD_MAX_DEVICES];  // device address of `scratch` on each device (set once)
std::mutex g_scratch_mu;
}  // namespace

// Resolves the device address of the scratch array on the current device, once per device (the
// name `scratch` in host code is only a stand-in, never a device address).  Called by mhd25_init.
int noalloc_setup(mhd25_ctx* c) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MHD_MAX_DEVICES) {
    c->err = "no-alloc setup: no current device";
    return -2;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch[dev]) return 0;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    c->err = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
    return -2;
  }
  g_scratch[dev] = (double*)ptr;
  return 0;
}

extern "C" int mhd25_rhs_magnetic_noalloc(mhd25_ctx* c, const double* rho, const double* u, const double* Bx,
                                          const double* By, const double* Bz, const double* eta, double* de,
                                          double* du, double* dBx, double* dBy, double* dBz) {
  if (!c || !rho || !u || !Bx || !By || !Bz || !de || !du || !dBx || !dBy || !dBz) return -1;
  const long K = c->mp.K, G = c->G;
  // the documented limit: the grids, and room for the element loads of W, N_x and N_y (no kernel writes those any
  // more; the accepted meshes stay what they were)
  const long a = c->m + 2, b = c->m + 1;
  const long need = 6 * G + K * (2 * a * b + a * a);
  if (need > MHD_NOALLOC_DOUBLES) {
    c->err = "rhs_magnetic_noalloc: the mesh needs " + std::to_string(need * 8) + " bytes of scratch, above the " +
             std::to_string(MHD_NOALLOC_DOUBLES * 8) + "-byte limit";
    return -1;
  }
  int dev = 0;
  double* ws = nullptr;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < MHD_MAX_DEVICES) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    ws = g_scratch[dev];
  }
  if (!ws) {
    c->err = "rhs_magnetic_noalloc: scratch not set up on the current device (create a context on it first)";
    return -2;
  }
  double* JE = ws;            // six grids: J_x, J_y, J_z, E_x, E_y, E_z
  if (const int r = mag_reconstruct_JE(c, u, Bx, By, Bz, eta, JE, c->opt.reduced_2d2v != 0)) return r;
  MagIO io{};
  io.rho = rho; io.us = u; io.bxs = Bx; io.bys = By; io.bzs = Bz;
  io.jx = JE; io.jy = JE + G; io.jz = JE + 2 * G;
  io.ex = JE + 3 * G; io.ey = JE + 4 * G; io.ez = JE + 5 * G;
  io.eta = eta;
  io.oe = de; io.ou = du; io.obx = dBx; io.oby = dBy; io.obz = dBz;
  return mag_update(c, io, 0);
}
