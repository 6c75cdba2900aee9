// Matrix-free SBM operator kernels for gfx950 (CDNA4, wave64).
//
//   brick_kernel    CG: one workgroup per brick of BX x BY x BZ background cells.  The
//                   brick's active cells (Alg. 1) are evaluated into an LDS copy of the
//                   brick's DoF lattice (on large operators a brick whose cells are all
//                   active by 1D line sweeps over the whole lattice; small ones and 3D p = 2
//                   and 3 cell by cell), with the rows of its surrogate-boundary faces
//                   (Alg. 3); points strictly inside the brick are
//                   then stored to v directly, points on the brick's boundary (shared with
//                   neighbouring bricks) go to halo slots that halo_reduce_kernel sums.
//   sbm_face_cg_kernel  CG surrogate-boundary faces (Alg. 3), before the bricks: (Rv, Rg)
//                   per face node, which the brick holding the face's cell expands and merges.
//   sbm_face_kernel DG surrogate-boundary faces (Alg. 3): (Rv, Rg) per face node.
//   dg_cell_kernel  DG: Laplace cell term plus the SIPG terms of the cell's interior faces,
//                   evaluated cell by cell (Alg. 2 split per side), plus the rows of the
//                   cell's surrogate faces; every cell writes only its own block.
//
// Every sum (cells into the brick lattice, face rows, brick-boundary planes, DG face rows) is
// taken in an order fixed by the setup, with no atomics: applies are bitwise reproducible.
//
// Work layout: an "entity" (cell or face) is handled by NP = (p+1)^(d-1) consecutive threads,
// EPB entities at a time per workgroup.  Thread t of an entity owns one pencil of p+1
// values along a coordinate axis; the (p+1)^d tile of the cell lives in LDS.  Within a
// cell, the p+1 DoFs along the first axis (an "x-run") are consecutive in both
// numberings, so gathers read p+1 consecutive entries from a per-run base index.
//
// Cell term in Kronecker-sum form: all active cells are translates of one reference cell
// with Jacobian h I (Sec. 3.4), so the Gauss-point loop of Alg. 1 is a fixed diagonal
// scaling and evaluate / quadrature / integrate collapse per axis into the 1D matrices
//   M_ij = sum_q w_q l_i(g_q) l_j(g_q),   K_ij = sum_q w_q l'_i(g_q) l'_j(g_q)
// (exact with p+1 Gauss points), A_K = h^(d-2) sum_k M x .. K(axis k) .. x M.  In 3D this
// is 7 one-dimensional sweeps instead of the 12 of the gradient form.
#include <algorithm>
#include <climits>
#include <cstring>
#include <type_traits>

#include "sbm_internal.h"

namespace sbm {
namespace {

template <int D, int N1>
struct Shape {
  static constexpr int NP = (D == 3) ? N1 * N1 : N1;
  static constexpr int NB = NP * N1;
};

// Entities per workgroup: fill up to 256 threads, keep the static LDS below ~60 KB.
template <typename T, int D, int N1, int NBUF, int EXTRA>
constexpr int epb() {
  constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  int e = 256 / NP;
  if (e < 1) e = 1;
  while (e > 1 && (e * NBUF * NB + 4 * e * NP + EXTRA) * (int)sizeof(T) > 60000) --e;
  return e;
}

// Entities per workgroup when there are few entities: one wavefront (at least one entity),
// so that small operators still spread over every CU.
template <typename T, int D, int N1, int NBUF>
constexpr int epb_one_wave() {
  constexpr int NP = Shape<D, N1>::NP, E = 64 / NP, F = epb<T, D, N1, NBUF, 0>();
  return E < 1 ? 1 : (E > F ? F : E);
}

// Workgroups that fill the device twice (two per compute unit).
inline int two_per_cu() {
  static const int n = [] {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                hipSuccess)
      return 512;
    return 2 * cus;
  }();
  return n;
}

// Brick of background cells per CG workgroup, chosen per degree so that the LDS lattice
// ((BX p + 1)(BY p + 1)(BZ p + 1) values) stays near 20 KB in FP64.
template <int D, int P, bool CELLS>
struct BrickDims {
  // 3D by p + 1 lanes per cell (CELLS, p <= 3): cells that fill whole wavefronts, 8x4x4, 7x6x4 and
  // 8x4x2 (shapes of half and twice the size measured within 3 % of these, at p=2 8 % slower at
  // half the size on a 150^3 mesh: more brick boundary); p=1 by sweeps 8x8x8
  // 3D, p >= 4: p=4,5 4x2x2, p=6 2x2x1, p=7 2x2x2, p=8 2x2x1 (at p=4, 4x2x2 measured faster than
  // 4x4x2, whose LDS allowed 3 workgroups per CU, and than 2x2x2; at p=6, 2x2x1 faster than 2x2x2
  // on a 48^3 mesh, which has too few 2x2x2 bricks to fill the device)
  // 2D: 8x8 up to p=2, 4x4 up to p=7, 3x3 for p=8 (a lattice row must fit 32 points)
  static constexpr int S3[9][3] = {{1, 1, 1}, {8, 8, 8}, {7, 6, 4}, {8, 4, 2}, {4, 2, 2},
                                   {4, 2, 2}, {2, 2, 1}, {2, 2, 2}, {2, 2, 1}};
  static constexpr bool SMALL = D == 3 && P == 1 && CELLS;  // 8x4x4
  static constexpr int BX = (D == 2) ? (P <= 2 ? 8 : (P <= 7 ? 4 : 3)) : S3[P][0];
  static constexpr int BY = (D == 2) ? BX : (SMALL ? 4 : S3[P][1]);
  static constexpr int BZ = (D == 2) ? 1 : (SMALL ? 4 : S3[P][2]);
};

// XCD-aware block order: the dispatcher hands block b to XCD (b mod 8), so give every XCD
// one contiguous range of logical blocks; neighbouring cells then share that XCD's L2.
__device__ __forceinline__ int xcd_block() {
  const int nb = gridDim.x;
  const int b = blockIdx.x;
  const int x = b & 7, k = b >> 3;
  const int per = nb >> 3, rem = nb & 7;
  return (x < rem) ? x * (per + 1) + k : rem * (per + 1) + (x - rem) * per + k;
}

__device__ __forceinline__ void atomic_add(double *p, double v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add(float *p, float v) { unsafeAtomicAdd(p, v); }

template <int N1>
__device__ __forceinline__ void lagrange_at(const double (&z)[N1], const double (&cinv)[N1], double x,
                                            double (&out)[N1]) {
  // l_j(x) = cinv_j prod_{m != j} (x - z_m), product form (stable when extrapolating)
  double dlt[N1], pre[N1], suf[N1];
#pragma unroll
  for (int m = 0; m < N1; ++m) dlt[m] = x - z[m];
  pre[0] = 1.0;
#pragma unroll
  for (int m = 1; m < N1; ++m) pre[m] = pre[m - 1] * dlt[m - 1];
  suf[N1 - 1] = 1.0;
#pragma unroll
  for (int m = N1 - 2; m >= 0; --m) suf[m] = suf[m + 1] * dlt[m + 1];
#pragma unroll
  for (int j = 0; j < N1; ++j) out[j] = cinv[j] * pre[j] * suf[j];
}

// ------------------------------------------------------------------------------------
// Cell term for one entity.  x: thread t's input pencil along the last axis (3D: t =
// i0 + N1 i1 holds u(i0, i1, k), k = 0..p; 2D: t = i0 holds u(i0, k)).  Returns in out
// the p+1 outputs of x-run t (3D: t = i1 + N1 i2; 2D: t = i1).  A, B: this entity's
// two (p+1)^d LDS tiles.  Contains barriers: every thread of the block must call it.
// ------------------------------------------------------------------------------------
// Even/odd pieces of a pencil: e_k = x_k + x_{p-k}, o_k = x_k - x_{p-k} (k < p+1 div 2),
// plus the middle value when p+1 is odd.
template <typename T, int N1>
struct EvenOdd {
  static constexpr int HC = (N1 + 1) / 2, HF = N1 / 2;
  T e[HC], o[HF > 0 ? HF : 1];
  __device__ __forceinline__ explicit EvenOdd(const T (&x)[N1]) {
#pragma unroll
    for (int k = 0; k < HF; ++k) {
      e[k] = x[k] + x[N1 - 1 - k];
      o[k] = x[k] - x[N1 - 1 - k];
    }
    if constexpr (N1 % 2 == 1) e[HF] = x[HF];
  }
};

// ye += E e, yo += O o for one centrosymmetric matrix given by its even/odd parts.
template <typename T, int N1>
__device__ __forceinline__ void eo_acc(const T *E, const T *O, const EvenOdd<T, N1> &v, T (&ye)[(N1 + 1) / 2],
                                       T (&yo)[N1 / 2 > 0 ? N1 / 2 : 1]) {
  constexpr int HC = (N1 + 1) / 2, HF = N1 / 2;
#pragma unroll
  for (int i = 0; i < HC; ++i)
#pragma unroll
    for (int k = 0; k < HC; ++k) ye[i] += E[i * HC + k] * v.e[k];
#pragma unroll
  for (int i = 0; i < HF; ++i)
#pragma unroll
    for (int k = 0; k < HF; ++k) yo[i] += O[i * HF + k] * v.o[k];
}

// y_i = ye_i + yo_i, y_{p-i} = ye_i - yo_i (and the middle row), times s.
template <typename T, int N1>
__device__ __forceinline__ void eo_combine(const T (&ye)[(N1 + 1) / 2], const T (&yo)[N1 / 2 > 0 ? N1 / 2 : 1],
                                           T s, T (&y)[N1]) {
  constexpr int HF = N1 / 2;
#pragma unroll
  for (int i = 0; i < HF; ++i) {
    y[i] = s * (ye[i] + yo[i]);
    y[N1 - 1 - i] = s * (ye[i] - yo[i]);
  }
  if constexpr (N1 % 2 == 1) y[HF] = s * ye[HF];
}

template <typename T, int N1>
struct EOAcc {
  T ye[(N1 + 1) / 2], yo[N1 / 2 > 0 ? N1 / 2 : 1];
  __device__ __forceinline__ EOAcc() {
#pragma unroll
    for (int i = 0; i < (N1 + 1) / 2; ++i) ye[i] = T(0);
#pragma unroll
    for (int i = 0; i < (N1 / 2 > 0 ? N1 / 2 : 1); ++i) yo[i] = T(0);
  }
};

template <typename T, int D, int N1>
__device__ __forceinline__ void kron_cell(const KTab<T, N1> &tab, int t, const T (&x)[N1], T *A, T *B, T scale,
                                          T (&out)[N1], bool on = true, bool work = true) {
  // on = false: compute but store nothing; work = false: only take part in the barriers (out
  // is left as it was)
  constexpr int NP = Shape<D, N1>::NP;
  if (work) {
    // last axis: a = M x, b = K x
    const EvenOdd<T, N1> ex(x);
    EOAcc<T, N1> ya, yb;
    eo_acc<T, N1>(tab.EM, tab.OM, ex, ya.ye, ya.yo);
    eo_acc<T, N1>(tab.EK, tab.OK, ex, yb.ye, yb.yo);
    T a[N1], b[N1];
    eo_combine<T, N1>(ya.ye, ya.yo, T(1), a);
    eo_combine<T, N1>(yb.ye, yb.yo, T(1), b);
    if (on) {
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        A[t + NP * i] = a[i];
        B[t + NP * i] = b[i];
      }
    }
  }
  __syncthreads();
  if constexpr (D == 3) {
    // pencils along axis 1; c = M a, e = K a + M b
    const int ix = t % N1, iz = t / N1;
    T a[N1], b[N1];
    if (work) {
#pragma unroll
      for (int j = 0; j < N1; ++j) {
        a[j] = A[ix + N1 * j + NP * iz];
        b[j] = B[ix + N1 * j + NP * iz];
      }
    }
    __syncthreads();
    if (work) {
      const EvenOdd<T, N1> ea(a), eb(b);
      EOAcc<T, N1> yc, ye;
      eo_acc<T, N1>(tab.EM, tab.OM, ea, yc.ye, yc.yo);
      eo_acc<T, N1>(tab.EK, tab.OK, ea, ye.ye, ye.yo);
      eo_acc<T, N1>(tab.EM, tab.OM, eb, ye.ye, ye.yo);
      T c[N1], e[N1];
      eo_combine<T, N1>(yc.ye, yc.yo, T(1), c);
      eo_combine<T, N1>(ye.ye, ye.yo, T(1), e);
      if (on) {
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          A[ix + N1 * i + NP * iz] = c[i];
          B[ix + N1 * i + NP * iz] = e[i];
        }
      }
    }
    __syncthreads();
  }
  if (work) {
    // pencils along axis 0 (thread t = run index); out = K c + M e
    T c[N1], e[N1];
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      c[j] = A[j + N1 * t];
      e[j] = B[j + N1 * t];
    }
    const EvenOdd<T, N1> ec(c), ee(e);
    EOAcc<T, N1> yo;
    eo_acc<T, N1>(tab.EK, tab.OK, ec, yo.ye, yo.yo);
    eo_acc<T, N1>(tab.EM, tab.OM, ee, yo.ye, yo.yo);
    eo_combine<T, N1>(yo.ye, yo.yo, scale, out);
  }
}

// Thread t's input pencil (see kron_cell) gathered through the x-run bases of a CG cell
// (cell_runs: the cell's (p+1)^(d-1) run bases, in LDS or in global memory).
template <typename T, int D, int N1>
__device__ __forceinline__ void gather_pencil(const int32_t *cell_runs, const T *__restrict__ u, int t, bool act,
                                              T (&x)[N1]) {
  const int i0 = (D == 3) ? t % N1 : t;
  const int r0 = (D == 3) ? t / N1 : 0;
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int run = (D == 3) ? r0 + N1 * k : k;
    x[k] = act ? u[cell_runs[run] + i0] : T(0);
  }
}

// ------------------------------------------------------------------------------------
// Face helpers (3D: tangential axes b < c; 2D: one tangential axis b)
// ------------------------------------------------------------------------------------
template <int D, int N1>
struct FaceAxes {
  int a, s, Sa, Sb, Sc;
  __device__ __forceinline__ FaceAxes(int code) {
    a = code >> 1;
    s = code & 1;
    Sa = (a == 0) ? 1 : (a == 1 ? N1 : N1 * N1);
    if (D == 3) {
      Sb = (a == 0) ? N1 : 1;        // lower tangential axis
      Sc = (a == 2) ? N1 : N1 * N1;  // upper tangential axis
    } else {
      Sb = (a == 0) ? N1 : 1;
      Sc = 0;
    }
  }
};

// Gauss -> GLL transposed interpolation of two face arrays f3, f4 (Gauss-point order
// qb + N1 qc), results at face node t = jb + N1 jc.  Uses f1, f2 as scratch.
template <typename T, int D, int N1>
__device__ __forceinline__ void face_integrate(const KTab<T, N1> &tab, int t, T *f1, T *f2, const T *f3,
                                               const T *f4, T &Rv, T &Rg) {
  if constexpr (D == 3) {
    const int qb = t % N1, jc = t / N1;
    T r1 = 0, r2 = 0;
#pragma unroll
    for (int qc = 0; qc < N1; ++qc) {
      r1 += tab.N[qc * N1 + jc] * f3[qb + N1 * qc];
      r2 += tab.N[qc * N1 + jc] * f4[qb + N1 * qc];
    }
    f1[t] = r1;
    f2[t] = r2;
    __syncthreads();
    const int jb = t % N1;
    T a1 = 0, a2 = 0;
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      a1 += tab.N[q * N1 + jb] * f1[q + N1 * jc];
      a2 += tab.N[q * N1 + jb] * f2[q + N1 * jc];
    }
    Rv = a1;
    Rg = a2;
  } else {
    T a1 = 0, a2 = 0;
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      a1 += tab.N[q * N1 + t] * f3[q];
      a2 += tab.N[q * N1 + t] * f4[q];
    }
    Rv = a1;
    Rg = a2;
  }
}

// GLL -> Gauss interpolation on the face of two node arrays f1, f2 (node order jb + N1 jc);
// returns the values at Gauss point t = qb + N1 qc.  Uses f3, f4 as scratch.
template <typename T, int D, int N1>
__device__ __forceinline__ void face_interpolate(const KTab<T, N1> &tab, int t, const T *f1, const T *f2,
                                                 T *f3, T *f4, T &o1, T &o2) {
  if constexpr (D == 3) {
    const int qb = t % N1, jc = t / N1;
    T r1 = 0, r2 = 0;
#pragma unroll
    for (int jb = 0; jb < N1; ++jb) {
      r1 += tab.N[qb * N1 + jb] * f1[jb + N1 * jc];
      r2 += tab.N[qb * N1 + jb] * f2[jb + N1 * jc];
    }
    f3[t] = r1;
    f4[t] = r2;
    __syncthreads();
    const int qc = t / N1;
    T a1 = 0, a2 = 0;
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      a1 += tab.N[qc * N1 + j] * f3[qb + N1 * j];
      a2 += tab.N[qc * N1 + j] * f4[qb + N1 * j];
    }
    o1 = a1;
    o2 = a2;
  } else {
    T a1 = 0, a2 = 0;
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      a1 += tab.N[t * N1 + j] * f1[j];
      a2 += tab.N[t * N1 + j] * f2[j];
    }
    o1 = a1;
    o2 = a2;
  }
}

// ------------------------------------------------------------------------------------
// One surrogate-boundary face (Alg. 3).  su: u_K in LDS (lexicographic), already synced.
// Returns Rv, Rg at this thread's face node t (face_row turns them into the (p+1)^d local
// rows).  xp: the shifted reference point of face Gauss point t, used only when act.
// f1..f4: NP values each of scratch.  Contains barriers.
//   dn u   = (2s-1)/h d/dxi_a u at the face Gauss points (sum factorisation),
//   E u    = u_K(xi_q), point evaluation with (p+1)^d terms per point,
//   tested:  w_q (sigma E u - dn u) against v, -w_q E u against dn v.
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1>
__device__ __forceinline__ void sbm_face_eval(const KTab<T, N1> &tab, const KScal &sc, int t, bool act,
                                              const FaceAxes<D, N1> &fa, const double (&xp)[D], const T *su,
                                              T *f1, T *f2, T *f3, T *f4, T &Rv, T &Rg) {
  constexpr int NP = Shape<D, N1>::NP;
  const T h = T(sc.h), sig = T(sc.sigma_gamma);
  const T sh = (fa.s ? T(1) : T(-1)) / h;  // normal sign over h
  const int jb = (D == 3) ? t % N1 : t, jc = (D == 3) ? t / N1 : 0;
  const int node_off = jb * fa.Sb + jc * fa.Sc;
  {
    T g = 0;
#pragma unroll
    for (int ia = 0; ia < N1; ++ia) g += (fa.s ? tab.D1[ia] : tab.D0[ia]) * su[ia * fa.Sa + node_off];
    f1[t] = g;
    f2[t] = g;
  }
  __syncthreads();
  T dn, dn2;
  face_interpolate<T, D, N1>(tab, t, f1, f2, f3, f4, dn, dn2);
  dn *= sh;

  T eu = 0, om = 0;
  if (act) {
    double l[D][N1];
#pragma unroll
    for (int k = 0; k < D; ++k) lagrange_at<N1>(tab.z, tab.cinv, xp[k], l[k]);
    T l0[N1], l1[N1];
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      l0[j] = T(l[0][j]);
      l1[j] = T(l[1][j]);
    }
    if constexpr (D == 3) {
#pragma unroll
      for (int i2 = 0; i2 < N1; ++i2) {
        T s1 = 0;
#pragma unroll
        for (int i1 = 0; i1 < N1; ++i1) {
          T s0 = 0;
#pragma unroll
          for (int i0 = 0; i0 < N1; ++i0) s0 += l0[i0] * su[i0 + N1 * i1 + NP * i2];
          s1 += l1[i1] * s0;
        }
        eu += T(l[2][i2]) * s1;
      }
      om = h * h * tab.w[t % N1] * tab.w[t / N1];
    } else {
#pragma unroll
      for (int i1 = 0; i1 < N1; ++i1) {
        T s0 = 0;
#pragma unroll
        for (int i0 = 0; i0 < N1; ++i0) s0 += l0[i0] * su[i0 + N1 * i1];
        eu += l1[i1] * s0;
      }
      om = h * tab.w[t];
    }
  }
  __syncthreads();  // f3/f4 reads of face_interpolate are done
  f3[t] = om * (sig * eu - dn);  // tested against v
  f4[t] = -om * eu * sh;         // tested against the reference derivative along a
  __syncthreads();
  face_integrate<T, D, N1>(tab, t, f1, f2, f3, f4, Rv, Rg);
}

// The face's result for the local row at position ia along the face normal, at this
// thread's face node: Rv on the face itself (ia = s p), plus Rg times the normal derivative
// of the 1D basis function ia at the face.
template <typename T, int D, int N1>
__device__ __forceinline__ T face_row(const KTab<T, N1> &tab, const FaceAxes<D, N1> &fa, int ia, T Rv, T Rg) {
  return ((ia == fa.s * (N1 - 1)) ? Rv : T(0)) + (fa.s ? tab.D1[ia] : tab.D0[ia]) * Rg;
}

// Brick description handed to the CG kernel.
struct BrickArgs {
  const int32_t *cell_off;   // n_bricks + 1
  const int32_t *runs;       // run bases of the active cells ((p+1)^(d-1) each), grouped by brick
  const int32_t *cell_loc;   // lattice offset of each cell's corner inside its brick
  // surrogate faces, numbered in brick order (a brick's faces are face_off[b] .. face_off[b+1])
  const int32_t *face_off;   // n_bricks + 1
  const int32_t *face_loc;   // lattice offset of each face's cell inside its brick
  const int32_t *face_code;  // per face: 2 axis + side
  const int32_t *cell_face;  // per cell: 64 x (first face of the cell, from the brick's first) + mask of codes
  const int32_t *row_base;   // n_bricks x rows: DoF id of the first globally present point
  const uint32_t *row_gmask; // bit x: lattice point x of the row is a DoF
  const uint32_t *row_bmask; // bit x: ... and is touched by an active cell of this brick
  // (halo indices) a row on the brick's y or z boundary: where its points 0 < x < LX - 1 start, less
  // one if its point x = 0 is a DoF, so that a point follows by its place among the row's DoFs
  const int32_t *row_hbase;
  const int32_t *row_hend;   // n_bricks x 2 x rows: the rows' points x = 0, then their points x = LX - 1
};

// One operator of a batch of applies (see the batched kernels after apply_impl): its arrays,
// vectors, scalars and its first workgroup in each stage's launch.
struct BatchItem {
  BrickArgs br;  // CG bricks
  const int32_t *face_code, *face_runs, *face_cell, *nbr, *halo_dof;
  const uint8_t *halo_mask;
  const double *face_xi;
  const void *u;
  void *v, *fbuf, *halo;
  KScal sc;
  int nf, nc, nh;
  int blk0[4];  // first workgroup of the item in each stage's launch
};

// A pointer that a kernel reads from memory or LDS is generic to the compiler: its loads and stores are
// flat ones, which wait on LDS too.
template <typename T>
using GlobalT = __attribute__((address_space(1))) T;

// The item of a workgroup of a batched kernel, its pointers marked global.
__device__ __forceinline__ BatchItem batch_item(const BatchItem *__restrict__ items, int i) {
  BatchItem it = items[i];
  auto global = [](auto *&p) {
    using P = std::remove_pointer_t<std::remove_reference_t<decltype(p)>>;
    p = (P *)(GlobalT<P> *)(uintptr_t)p;  // (the compiler drops a cast there and back)
  };
  global(it.br.cell_off);
  global(it.br.runs);
  global(it.br.cell_loc);
  global(it.br.face_off);
  global(it.br.face_loc);
  global(it.br.face_code);
  global(it.br.cell_face);
  global(it.br.row_base);
  global(it.br.row_gmask);
  global(it.br.row_bmask);
  global(it.br.row_hbase);
  global(it.br.row_hend);
  global(it.face_code);
  global(it.face_runs);
  global(it.face_cell);
  global(it.nbr);
  global(it.halo_dof);
  global(it.halo_mask);
  global(it.face_xi);
  global(it.u);
  global(it.v);
  global(it.fbuf);
  global(it.halo);
  return it;
}

// ------------------------------------------------------------------------------------
// CG brick kernel
// ------------------------------------------------------------------------------------
// Geometry of the CG brick kernel by sweeps for (D, P): lattice extents, block size (enough threads
// for the longest set of lattice lines, at most 256 so that several workgroups share a CU),
// cells per batch on the per-cell path, and the LDS size (the larger of the two paths,
// which share one buffer).
template <typename T, int D, int N1>
struct SweepBrickCfg {
  static constexpr int P = N1 - 1, NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  static constexpr int BX = BrickDims<D, P, false>::BX, BY = BrickDims<D, P, false>::BY,
                       BZ = BrickDims<D, P, false>::BZ;
  static constexpr int LX = BX * P + 1, LY = BY * P + 1, LZ = (D == 3) ? BZ * P + 1 : 1;
  static constexpr int NL = LX * LY * LZ, NROWS = LY * LZ;
  static constexpr int LINES = (D == 3) ? ((LX * LY > LX * LZ ? LX * LY : LX * LZ) > LY * LZ
                                               ? (LX * LY > LX * LZ ? LX * LY : LX * LZ)
                                               : LY * LZ)
                                        : (LX > LY ? LX : LY);
  static constexpr int NT0 = ((LINES + 63) / 64) * 64;
  // (3D p=4: 192 threads measured faster than 256 and 320 in both precisions: FP32 brick kernel
  // 21.1 / 21.9 / 25.9 us, FP64 28.5 / 29.8 / 36.0 us)
  static constexpr int NT = NT0 < 128 ? 128 : (NT0 > 256 ? 256 : NT0);
  static constexpr int EPB0 = NT / NP;
  static constexpr int EPB = EPB0 < 1 ? 1 : EPB0;   // faces per batch (and thread groups with NP threads)
  static constexpr int NG = (NT + NP - 1) / NP;      // thread groups (the last may be partial)
  // cells per batch of the per-cell path: each has two tiles of NB values; the groups beyond
  // only take part in the barriers.  At 3D p=4 the batch is cut to 4 cells so that the tiles
  // and the staged run bases fit in the sweep arrays' space.
  static constexpr int EPC0 = (D == 3 && P == 4) ? 4 : EPB;  // (FP32 too: 20.3 against 20.9 us)
  static constexpr int EPC = EPC0 < EPB ? EPC0 : EPB;
  static constexpr int NTILE = EPC;  // tile pairs (the other groups store nothing)
  // LDS in elements of T: the lattice accumulator (the cell and face rows are summed into it in
  // the apply's precision, in a fixed order), then either the second sweep array of the full
  // path (the first one is the accumulator itself) or the per-cell tiles.
  static constexpr int MAXC = BX * BY * BZ;  // cells of a full brick
  static constexpr int TAIL_SWEEP = NL;
  // per-cell path: the tiles, then (where they are small: p >= 4 in 3D) the brick's run
  // bases and cell offsets (int32), staged in one round trip instead of read per batch
  static constexpr int RUNS_B = (MAXC * NP + MAXC) * 4;
  static constexpr bool STAGE_RUNS = RUNS_B <= 2560;
  static constexpr int RUNS_T = STAGE_RUNS ? (RUNS_B + (int)sizeof(T) - 1) / (int)sizeof(T) : 0;
  // ... then the partial brick's row masks (a full brick's are all ones)
  static constexpr int MASK_T = (2 * NROWS * 4 + (int)sizeof(T) - 1) / (int)sizeof(T);
  static constexpr int TAIL_CELLS = 2 * NTILE * NB + RUNS_T + MASK_T;
  static constexpr int SMEM = NL + (TAIL_SWEEP > TAIL_CELLS ? TAIL_SWEEP : TAIL_CELLS);
};

// Form of an operator's brick kernel: cell by cell up to kCellsMax cells, lattice sweeps
// (sweeps_body) above.  Cell by cell means p + 1 lanes per cell in 3D at p <= 3 (cells_body), else
// (p+1)^(d-1) threads per cell (tile_body).
// 3D, p = 2 and 3: always; the lanes' results leave four or more wavefronts per SIMD (p=3, 96^3: 52
// against 73 us FP64; 24^3: 11 against 24 us FP32.  At p=4 the lanes, FP64 160 registers and 1 KB of
// LDS per cell, and the sweeps measured alike on 64^3).
// 3D, p = 1: the lanes' smaller bricks leave more DoFs on brick boundaries (51 % against 33 %), which
// decides once the device is full several times over (FP64 / FP32 apply of 2.4 M cells 79 / - against
// 113 us, of 5.7 M 158 / 125 against 155 / 116, of 9.6 M 254 / 197 against 226 / 150).
// 3D, p >= 4, and 2D: all cells at once is one short chain (one gather, one pass per axis, one
// write-out) where the sweeps of a brick with cut cells run batch after batch; that decides as long
// as every brick has a place on the device, and the larger LDS and workgroup against it after that.
// Brick kernel alone, sweeps -> cells in us, balls of radius 0.75 in [-1,1]^3, FP64 and FP32:
//   p=4  24^3 17.1 -> 10.5, 15.9 ->  9.5   40^3 21.0 -> 18.9, 16.8 -> 15.4   48^3 23.3 -> 25.2, 19.2 -> 20.9
//   p=5  24^3 18.9 -> 12.1, 16.7 -> 10.7   32^3 22.1 -> 18.6, 17.7 -> 12.6   40^3 26.6 -> 31.0, 20.5 -> 24.4
//   p=6  16^3 14.6 -> 11.6, 11.2 ->  9.8   24^3 16.8 -> 14.5, 12.1 -> 11.2   48^3 58.9 -> 58.4, 28.0 -> 34.3
//   p=7  12^3 21.2 -> 13.1, 16.1 -> 11.6   20^3 18.4 -> 14.8, 15.0 -> 12.3   30^3 33.1 -> 30.8, 21.5 -> 19.2
//   p=8  12^3 18.7 -> 13.6, 13.8 -> 12.1   20^3 21.0 -> 17.1, 15.5 -> 14.4   36^3 74.1 -> 64.0, 31.6 -> 40.8
// (the balls hold about 0.22 n^3 cells); 2D, FP64 and FP32:
//   p=2  16^2 10.8 ->  9.9, 10.4 ->  9.2   p=6 300^2 16.3 -> 15.3, 13.0 -> 12.0   p=8 200^2 19.2 -> 16.1, 12.9 -> 11.7
//   p=4 512^2 17.7 -> 18.3, 13.8 -> 15.9   p=5 400^2 17.2 -> 18.1, 13.0 -> 15.0   p=8 600^2 91 -> 106, 48 -> 62
// The form is fixed at setup, so one line holds for both precisions: below the first size at which either
// loses, which in 3D is FP32 (p=8 at 36^3 would gain 14 % by cells in FP64 and lose 29 % in FP32).  It is
// drawn in cells, which the caller knows: 16,384 cells are about 1,100 bricks at 3D p=4, 4,096 about 1,100
// at p=6.  All degrees of 2D share one line, below the first that loses (p=4); p=6 at 300^2 and p=8 at 200^2
// would still gain 6 to 16 %.
constexpr int64_t kAll = INT64_MAX;
constexpr int64_t kCellsMax[2][9] = {{0, 16384, 16384, 16384, 16384, 16384, 16384, 16384, 16384},
                                     {0, (int64_t)1 << 22, kAll, kAll, 16384, 8192, 4096, 8192, 4096}};
template <int D, int N1>
constexpr bool has_sweeps() {
  return kCellsMax[D - 2][N1 - 1] != kAll;
}

// Bricks by cell places, (p+1)^(d-1) threads each, all at once or (SPLIT > 1) a part of the brick's cells
// at a time
template <typename T, int D, int N1, int SPLIT = 1>
struct TileBrickCfg {
  static constexpr int DIM = D, P = N1 - 1, NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  static constexpr int BX = BrickDims<D, P, false>::BX, BY = BrickDims<D, P, false>::BY,
                       BZ = BrickDims<D, P, false>::BZ;
  static constexpr int LX = BX * P + 1, LY = BY * P + 1, LZ = (D == 3) ? BZ * P + 1 : 1, NROWS = LY * LZ;
  static constexpr int MAXC = BX * BY * BZ, PASS = MAXC / SPLIT;
  static constexpr int NW = (PASS * NP + 63) / 64, NT = 64 * NW;
  static constexpr int TILE = NB;
};

// SPLIT of a batch of many bricks by cells (1: none), and the bricks that it takes.  3D p=4 and 5: all
// at once four and three bricks are on a CU, and a batch of several times as many is slower than it was
// by sweeps, which a batch may not take as its results are those of the single applies.  Prepared
// batches of 16 balls, us by sweeps / by cells at once / in four parts, FP64 and FP32:
//   p=4  1,220 bricks  44 / 41 / 45   35 / 33 / 36    3,475  77 / 79 / 79   57 / 61 / 58    8,167  134 / 146 / 135   87 / 106 /  89
//   p=5  1,220 bricks  67 / 64 / 62   42 / 43 / 42    2,035  89 / 93 / 83   59 / 62 / 60    5,499  186 / 210 / 166  100 / 120 / 102
// (p=6, in two parts: 8,200 bricks 155 / 151 / 167 and 89 / 92 / 97; p=7 and 8 are faster at once at any size.)
template <int D, int N1>
constexpr int tile_split() {
  return D == 3 && (N1 == 5 || N1 == 6) ? 4 : 1;
}
template <typename T, int N1>
constexpr int tile_split_from() {
  return N1 == 5 ? (sizeof(T) == 8 ? 4096 : 2048) : 1024;
}

template <typename T, int N1>
struct CellBrickCfg {
  static constexpr int DIM = 3, D = 3, P = N1 - 1, NP = N1 * N1, NB = NP * N1;
  static constexpr int BX = BrickDims<D, P, true>::BX, BY = BrickDims<D, P, true>::BY,
                       BZ = BrickDims<D, P, true>::BZ;
  static constexpr int LX = BX * P + 1, LY = BY * P + 1, LZ = BZ * P + 1, NROWS = LY * LZ;
  static constexpr int MAXC = BX * BY * BZ;
  static constexpr int CPW = 64 / N1;                    // cells per wavefront
  static constexpr int NW = (MAXC + CPW - 1) / CPW, NT = 64 * NW;
  // The transposes between x-runs and y-lines: four planes in flight per wavefront, plane-major,
  // cells SC apart.  They use the LDS of the wavefront's share of the
  // cells' (p+1)^3 results, which follow.  (The strides with the fewest LDS bank conflicts.)
  static constexpr int SC = N1 == 4 ? 17 : NP;
  static constexpr int TILE = (NB > 4 * SC ? NB : 4 * SC) | (N1 == 4 ? 0 : 1);
};

template <typename T, int D, int N1, bool CELLS>
struct BrickCfg
    : std::conditional_t<!CELLS, SweepBrickCfg<T, D, N1>,
                         std::conditional_t<D == 3 && N1 <= 4, CellBrickCfg<T, N1>, TileBrickCfg<T, D, N1>>> {};

// Lattice-line segments of a full brick.  A line of B cells has B p + 1 nodes; the segment of
// cell j is nodes j p .. j p + p, and neighbouring segments share one node.  One lane per
// segment, the B lanes of a line side by side in a group of G = pow2 >= B lanes of one
// wavefront: each lane forms its cell's p + 1 outputs, takes the previous lane's last output
// for its first node (the sum of both cells' rows there), and stores nodes j p .. j p + p - 1
// (the last lane also node B p).  Every input is read before any lane of the line stores.
template <int G, typename T>
__device__ __forceinline__ T from_prev_lane(T y, int j) {
  if constexpr (G == 1) {
    return T(0);
  } else {
    const T w = __shfl_up(y, 1, G);
    return j > 0 ? w : T(0);
  }
}

template <int B>
struct LaneGroup {
  static constexpr int G = B <= 1 ? 1 : (B <= 2 ? 2 : (B <= 4 ? 4 : (B <= 8 ? 8 : 16)));
  static_assert(B <= 16 && 64 % G == 0, "segment groups must tile a wavefront");
};

template <typename T, int D, int N1>
__device__ __forceinline__ void sweeps_body(const int blk, BrickArgs br, const T *__restrict__ fbuf,
                                           const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
                                           int nhalo, KTab<T, N1> tab, T scale, int parts) {
  using C = SweepBrickCfg<T, D, N1>;
  constexpr int P = C::P, NP = C::NP, NB = C::NB, EPB = C::EPB;
  constexpr int BX = C::BX, BY = C::BY, BZ = C::BZ, LX = C::LX, LY = C::LY, LZ = C::LZ;
  constexpr int NL = C::NL, NROWS = C::NROWS;
  static_assert(LX <= 32, "row masks hold 32 points");
  __shared__ T smem[C::SMEM];
  T *const acc = smem;             // the brick lattice (both paths)
  T *const tail = smem + NL;       // per-cell tiles, or the second sweep array
  const int brick = blk;
  const int tid = threadIdx.x;
  constexpr int nthr = C::NT;  // the launch uses exactly NT threads
  const int le = tid / NP, t = tid - le * NP;
  const int64_t rb = (int64_t)brick * NROWS;
  // lattice offset of thread t's x-run inside a cell tile
  const int run_off = (D == 3) ? (t % N1) * LX + (t / N1) * LX * LY : t * LX;
  const int c0 = br.cell_off[brick], c1 = br.cell_off[brick + 1];
  const int f0 = br.face_off[brick], f1e = br.face_off[brick + 1];
  const bool full = (c1 - c0) == C::MAXC;
  // Everything that does not depend on u is fetched in one round trip at the start: the
  // brick's row descriptors (every later lattice access indexes them), for a partial brick
  // its cells' run bases and lattice offsets, and the first batch of surrogate-face results
  // (held in registers through the cell phase).
  __shared__ int32_t s_base[NROWS], s_hbase[NROWS];
  // (the partial brick's run bases, cell offsets and row masks sit behind the per-cell tiles;
  // a full brick's rows are all DoFs, all touched by its cells: masks of all ones, not stored,
  // which keeps the static LDS small enough for one more workgroup per CU)
  int32_t *const s_runs = reinterpret_cast<int32_t *>(tail + 2 * C::NTILE * NB);
  int32_t *const s_loc = s_runs + C::MAXC * NP;
  uint32_t *const s_gmask = reinterpret_cast<uint32_t *>(tail + 2 * C::NTILE * NB + C::RUNS_T);
  uint32_t *const s_bmask = s_gmask + NROWS;
  for (int r = tid; r < NROWS; r += nthr) {
    s_base[r] = br.row_base[rb + r];
    s_hbase[r] = br.row_hbase[rb + r];
    if (!full) {
      s_gmask[r] = br.row_gmask[rb + r];
      s_bmask[r] = br.row_bmask[rb + r];
    }
  }
  constexpr int NE = (2 * NROWS + nthr - 1) / nthr;  // row ends per thread
  int32_t hend[NE];
#pragma unroll
  for (int m = 0; m < NE; ++m) {
    const int i = tid + m * nthr;
    hend[m] = br.row_hend[2 * rb + (i < 2 * NROWS ? i : 0)];
  }
  if (C::STAGE_RUNS && !full && (parts & SBM_PART_CELLS)) {
    for (int i = tid; i < (c1 - c0) * NP; i += nthr) s_runs[i] = br.runs[(int64_t)c0 * NP + i];
    for (int i = tid; i < c1 - c0; i += nthr) s_loc[i] = br.cell_loc[c0 + i];
  }
  // a cell's run bases and lattice offset (by the cell's rank inside the brick)
  const int32_t *const runs_of = C::STAGE_RUNS ? s_runs : br.runs + (int64_t)c0 * NP;
  const int32_t *const loc_of = C::STAGE_RUNS ? s_loc : br.cell_loc + c0;
  const bool do_faces = (parts & SBM_PART_SBM_FACES) != 0;
  int fcode = 0, floc = 0;
  T fRv = T(0), fRg = T(0);
  if (do_faces && le < EPB && f0 + le < f1e) {
    const int f = f0 + le;
    fcode = br.face_code[f];
    floc = br.face_loc[f];
    fRv = fbuf[(int64_t)f * 2 * NP + t];
    fRg = fbuf[(int64_t)f * 2 * NP + NP + t];
  }
  __syncthreads();

  if (full && (parts & SBM_PART_CELLS)) {
    // ---- full brick: the sum of the cell operators over a tensor-product block of cells is
    // the Kronecker sum of the 1D operators assembled along each direction; sweep the
    // brick lattice line by line (a = M u, b = K u along the last axis, then c = M a,
    // e = K a + M b, then h (K c + M e)), in place in LDS. ----
    // sweep arrays: a/c in the accumulator itself (the last sweep writes in place), b/e in the
    // tail
    T *const LA = acc;
    T *const LB = tail;
    // last axis (z in 3D, y in 2D): a = M u, b = K u, gathered from u (every point of a full
    // brick is a DoF: id = row base + x)
    {
      constexpr int NC = (D == 3) ? BZ : BY, G = LaneGroup<NC>::G;
      constexpr int NLINE = (D == 3) ? LX * LY : LX;
      // every thread's segments are loaded before any is swept: one round trip to memory
      constexpr int NQ = (NLINE * G + nthr - 1) / nthr;
      T xus[NQ][N1];
#pragma unroll
      for (int r = 0; r < NQ; ++r) {
        const int q = tid + r * nthr;
        const int j = q % G, line = q / G;
        const int x = line % LX, y = (D == 3) ? line / LX : 0;
        const bool live = q < NLINE * G && j < NC;
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          const int row = (D == 3) ? y + LY * (j * P + i) : (j * P + i);
          xus[r][i] = live ? u[s_base[live ? row : 0] + x] : T(0);
        }
      }
#pragma unroll
      for (int r = 0; r < NQ; ++r) {
        const int q = tid + r * nthr;
        const int j = q % G, line = q / G;
        const int x = line % LX, y = (D == 3) ? line / LX : 0;
        const bool live = q < NLINE * G && j < NC;
        T ya[N1], yb[N1];
        {
          const EvenOdd<T, N1> ex(xus[r]);
          EOAcc<T, N1> aa, ab;
          eo_acc<T, N1>(tab.EM, tab.OM, ex, aa.ye, aa.yo);
          eo_acc<T, N1>(tab.EK, tab.OK, ex, ab.ye, ab.yo);
          eo_combine<T, N1>(aa.ye, aa.yo, T(1), ya);
          eo_combine<T, N1>(ab.ye, ab.yo, T(1), yb);
        }
        ya[0] += from_prev_lane<G>(ya[P], j);
        yb[0] += from_prev_lane<G>(yb[P], j);
        if (live) {
          const int pt0 = (D == 3) ? x + LX * (y + LY * (j * P)) : x + LX * (j * P);
          constexpr int SL = (D == 3) ? LX * LY : LX;
#pragma unroll
          for (int i = 0; i < P; ++i) {
            LA[pt0 + i * SL] = ya[i];
            LB[pt0 + i * SL] = yb[i];
          }
          if (j == NC - 1) {
            LA[pt0 + P * SL] = ya[P];
            LB[pt0 + P * SL] = yb[P];
          }
        }
      }
    }
    __syncthreads();
    if constexpr (D == 3) {
      // y: c = M a, e = K a + M b, in place
      constexpr int G = LaneGroup<BY>::G;
      for (int q = tid; q < LX * LZ * G; q += nthr) {
        const int j = q % G, line = q / G;
        const int x = line % LX, z = line / LX;
        const bool live = j < BY;
        const int o = x + LX * LY * z + j * P * LX;
        T xa[N1], xb[N1], yc[N1], ye[N1];
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          xa[i] = live ? LA[o + i * LX] : T(0);
          xb[i] = live ? LB[o + i * LX] : T(0);
        }
        {
          const EvenOdd<T, N1> ea(xa), eb(xb);
          EOAcc<T, N1> ac, ae;
          eo_acc<T, N1>(tab.EM, tab.OM, ea, ac.ye, ac.yo);
          eo_acc<T, N1>(tab.EK, tab.OK, ea, ae.ye, ae.yo);
          eo_acc<T, N1>(tab.EM, tab.OM, eb, ae.ye, ae.yo);
          eo_combine<T, N1>(ac.ye, ac.yo, T(1), yc);
          eo_combine<T, N1>(ae.ye, ae.yo, T(1), ye);
        }
        yc[0] += from_prev_lane<G>(yc[P], j);
        ye[0] += from_prev_lane<G>(ye[P], j);
        if (live) {
#pragma unroll
          for (int i = 0; i < P; ++i) {
            LA[o + i * LX] = yc[i];
            LB[o + i * LX] = ye[i];
          }
          if (j == BY - 1) {
            LA[o + P * LX] = yc[P];
            LB[o + P * LX] = ye[P];
          }
        }
      }
      __syncthreads();
    }
    // x: out = h (K c + M e), written over c
    {
      constexpr int G = LaneGroup<BX>::G;
      for (int q = tid; q < NROWS * G; q += nthr) {
        const int j = q % G, row = q / G;
        const bool live = j < BX;
        const int o = LX * row + j * P;
        T xc[N1], xe[N1], yo[N1];
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          xc[i] = live ? LA[o + i] : T(0);
          xe[i] = live ? LB[o + i] : T(0);
        }
        {
          const EvenOdd<T, N1> ec(xc), ee(xe);
          EOAcc<T, N1> ao;
          eo_acc<T, N1>(tab.EK, tab.OK, ec, ao.ye, ao.yo);
          eo_acc<T, N1>(tab.EM, tab.OM, ee, ao.ye, ao.yo);
          eo_combine<T, N1>(ao.ye, ao.yo, scale, yo);
        }
        yo[0] += from_prev_lane<G>(yo[P], j);
        if (live) {
#pragma unroll
          for (int i = 0; i < P; ++i) acc[o + i] = yo[i];
          if (j == BX - 1) acc[o + P] = yo[P];
        }
      }
    }
    __syncthreads();
  } else {
    for (int i = tid; i < NL; i += nthr) acc[i] = T(0);
    __syncthreads();
  }

  if (!full && (parts & SBM_PART_CELLS)) {
    // ---- partial brick: cell by cell (EPC cells per batch; the other thread groups only
    // take part in the barriers) ----
    constexpr int EPC = C::EPC, NTILE = C::NTILE;
    const bool grp = le < EPC;
    const int tl = grp ? le : 0;  // groups beyond EPC only take part in the barriers
    T *A = tail + tl * NB, *B = tail + NTILE * NB + tl * NB;
    // software pipeline: the pencils of batch b+1 are in flight while batch b computes
    T x[N1];
    {
      const bool act = grp && c0 + le < c1;
      gather_pencil<T, D, N1>(runs_of + (act ? le : 0) * NP, u, t, act, x);
    }
    for (int b = c0; b < c1; b += EPC) {
      const int idx = b + le;
      const bool act = grp && idx < c1;
      const int loc = act ? loc_of[idx - c0] : 0;
      const int idn = idx + EPC;
      const bool actn = grp && idn < c1;
      T xn[N1], out[N1];
      gather_pencil<T, D, N1>(runs_of + (actn ? idn - c0 : 0) * NP, u, t, actn, xn);
      kron_cell<T, D, N1>(tab, t, x, A, B, scale, out, grp, grp);
#pragma unroll
      for (int i = 0; i < N1; ++i) x[i] = xn[i];
      // the batch's cells add their rows in slot order (a cell's runs are disjoint), so every
      // lattice point sums its cells in the same order on every launch: bitwise reproducible
      const int nslot = (c1 - b) < EPC ? (c1 - b) : EPC;
      for (int k = 0; k < nslot; ++k) {
        if (le == k) {
#pragma unroll
          for (int i = 0; i < N1; ++i) acc[loc + run_off + i] += out[i];
        }
        __syncthreads();
      }
    }
  }
  if (do_faces) {
    // ---- the brick's surrogate faces: sbm_face_cg_kernel left (Rv, Rg) per face node in
    // fbuf; expand them into the (p+1)^d local rows and add those into the lattice.  The
    // batch's data is in registers (the first batch since the start); the next batch's is
    // fetched while this one merges. ----
    constexpr int SL1 = LX, SL2 = LX * LY;  // lattice strides of axes 1 and 2
    for (int b = f0; b < f1e; b += EPB) {
      const int f = b + le;
      const bool fact = le < EPB && f < f1e;
      const int fn = f + EPB;
      int ncode = 0, nloc = 0;
      T nRv = T(0), nRg = T(0);
      if (le < EPB && fn < f1e) {
        ncode = br.face_code[fn];
        nloc = br.face_loc[fn];
        nRv = fbuf[(int64_t)fn * 2 * NP + t];
        nRg = fbuf[(int64_t)fn * 2 * NP + NP + t];
      }
      int node = 0, Sa = 0;
      T row[N1];
      if (fact) {
        const FaceAxes<D, N1> fa(fcode);
        const int loc = floc;
        const T Rv = fRv, Rg = fRg;
        const int a = fa.a;
        const int jb = (D == 3) ? t % N1 : t, jc = (D == 3) ? t / N1 : 0;
        // normal axis a; tangential axes in increasing order (b < c), as in FaceAxes
        Sa = (a == 0) ? 1 : (a == 1 ? SL1 : SL2);
        const int Sb = (a == 0) ? SL1 : 1;
        const int Sc = (D == 3) ? ((a == 2) ? SL1 : SL2) : 0;
        node = loc + jb * Sb + jc * Sc;
#pragma unroll
        for (int ia = 0; ia < N1; ++ia) row[ia] = face_row<T, D, N1>(tab, fa, ia, Rv, Rg);
      }
      // faces add in slot order (one face's node lines are disjoint): reproducible sums
      const int nslot = (f1e - b) < EPB ? (f1e - b) : EPB;
      for (int k = 0; k < nslot; ++k) {
        if (fact && le == k) {
#pragma unroll
          for (int ia = 0; ia < N1; ++ia) acc[node + ia * Sa] += row[ia];
        }
        __syncthreads();
      }
      fcode = ncode;
      floc = nloc;
      fRv = nRv;
      fRg = nRg;
    }
  }
  __syncthreads();
  // write-out: points strictly inside the brick box belong to this brick alone: final value.  Points
  // on the box boundary go to plane k = [x == 0] + 2 [y == 0] + 4 [z == 0] of the halo (the
  // brick's side of the point; bricks sharing the point differ in k), at the point's halo
  // index; halo_reduce_kernel sums the planes.
  // The points 0 < x < LX - 1, x fastest: stores are row-contiguous.  Each wavefront takes RPW whole
  // rows per pass, so a lane's x is fixed, and a pass only advances the row; (y, z) of the row
  // advance by a constant.  The passes are unrolled, every LDS read first, so that one wait covers
  // them all.
  {
    constexpr int W = LX - 2, RPW = 64 / W, NW = C::NT / 64, STEP = NW * RPW;
    constexpr int NPASS = (NROWS + STEP - 1) / STEP;
    constexpr int QY = STEP % LY, QZ = STEP / LY;
    static_assert(RPW >= 1 && C::NT % 64 == 0, "a wavefront holds at least one lattice row");
    const int lane = tid & 63, rl = lane / W, x = 1 + lane - rl * W;
    const bool xl = rl < RPW;
    const uint32_t below = (1u << x) - 1u;
    const int row0 = (tid >> 6) * RPW + rl;
    int y = row0 % LY, z = row0 / LY;
    constexpr int CH = NPASS < 9 ? NPASS : 9;  // passes per group (bounds the registers held)
#pragma unroll
    for (int k0 = 0; k0 < NPASS; k0 += CH) {
      T val[CH];
      int base[CH], hb[CH];
      uint32_t gmk[CH], bmk[CH];
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        const int row = row0 + (k0 + k) * STEP;
        const bool on = xl && k0 + k < NPASS && row < NROWS;
        const int rc = on ? row : 0;
        val[k] = acc[rc * LX + x];
        base[k] = s_base[rc];
        hb[k] = s_hbase[rc];
        gmk[k] = full ? ~0u : s_gmask[rc];
        bmk[k] = (full || !on) ? (on ? ~0u : 0u) : s_bmask[rc];
      }
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        const bool brow = ((unsigned)(y - 1) >= (unsigned)(LY - 2)) |
                          ((D == 3) & ((unsigned)(z - 1) >= (unsigned)(LZ - 2)));
        const int plane = (y == 0 ? 2 : 0) | ((D == 3 && z == 0) ? 4 : 0);
        T *dst = (brow ? halo + ((int64_t)plane * nhalo + hb[k]) : v + base[k]) + __popc(gmk[k] & below);
        if ((bmk[k] >> x) & 1u) *dst = val[k];
        y += QY;
        z += QZ;
        if (y >= LY) {
          y -= LY;
          ++z;
        }
      }
    }
  }
  // The rows' ends: y fastest, as their halo indices.  (Ahead of the rows' other points they held up the
  // stores of large 2D operators: 3692^2 Q1 FP32 apply 71.5 against 66.6 us, 1230^2 Q3 44.5 against 43.0.)
#pragma unroll
  for (int m = 0; m < NE; ++m) {
    const int i = tid + m * nthr, side = i >= NROWS ? 1 : 0, r = i < 2 * NROWS ? i - side * NROWS : 0;
    const int y = r % LY, z = r / LY, x = side ? LX - 1 : 0;
    const uint32_t bm = full ? ~0u : s_bmask[r];
    const int plane = (side ? 0 : 1) | (y == 0 ? 2 : 0) | ((D == 3 && z == 0) ? 4 : 0);
    const T val = acc[r * LX + x];
    if (i < 2 * NROWS && ((bm >> x) & 1u)) halo[(int64_t)plane * nhalo + hend[m]] = val;
  }
}

// ------------------------------------------------------------------------------------
// Bricks of 3D cells of low degree (p <= 3): p + 1 lanes per cell, every cell on its own.
// Lane j of a cell sweeps x-run j of a plane in registers, turns the plane over through LDS
// (within its wavefront: no barrier), sweeps y-line j, and keeps the p + 1 planes' z sums of its
// y-line, (p+1)^2 results, in registers; it adds the rows of the cell's surrogate faces there.  The
// cells' results go to LDS once, and every lattice point then sums its cells' values as it is
// stored.
// What bounds it: the latency of a brick's phases on small meshes, and with the device full half of
// the HBM rate (150^3 Q2 FP64, 5.8 M DoFs).  The lattice sweeps, which take a brick with a missing
// cell batch by batch with a barrier for each cell and each face of a batch, spent their time in
// those bricks: these have up to 168 cells, and small meshes hold no others.  Whole apply replayed from a
// graph, by sweeps -> now: 45^3 Q2 FP32 31.4 -> 12.2 us; 30^3 Q1 FP64 73.2 -> 10.7; 96^3 Q3 FP64 86.1 ->
// 64.4; 150^3 Q2 FP64 84.7 -> 77.9.  The x-runs' first DoFs come from the row descriptors: reading them from
// the cells' table cost 36 B per cell at p=2, 5 % of the kernel.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Keeps the computation of x ahead of the branch that follows (LDS reads would sink into it one by
// one).
template <typename T>
__device__ __forceinline__ void settle(T &x) {
  asm volatile("" : "+v"(x));
}

// Rows of a brick's lattice in LDS, sorted by kind (y and z inside a cell, z inside and y on a plane
// between cells, y inside and z on such a plane, both on planes; in 2D there is the one plane z = 0).
template <typename T, class C>
struct BrickRows {
  static constexpr int P = C::P, YI = C::BY * (P - 1), ZI = C::DIM == 3 ? C::BZ * (P - 1) : 0, YB = C::BY + 1,
                       ZB = C::DIM == 3 ? C::BZ + 1 : 1;
  static constexpr int K1 = YI * ZI, K2 = K1 + YB * ZI, K3 = K2 + YI * ZB;  // first row of each kind but the first
  static_assert(K3 + YB * ZB == C::NROWS, "every row once");
  static_assert(C::NROWS <= C::NT, "one row per thread");
  static_assert(C::LX <= 32, "row masks hold 32 points");
  enum { kLowY = 1, kHighY = 2, kLowZ = 4, kHighZ = 8, kY0 = 16, kZ0 = 32 };
  T *dst[C::NROWS];           // where the points 0 < x < LX-1 go, by their place among the row's DoFs
  int32_t off[C::NROWS];      // 256 x (place of the row in the results) + flags
  uint32_t gmask[C::NROWS], bmask[C::NROWS];
  int32_t base[C::NROWS];     // by the row's own place y + LY z: id of its first DoF,
  uint32_t first[C::NROWS];   // mask of its DoFs

  // One row per thread (full: all masks are ones).  A barrier has to follow.  The halo indices of the
  // row's ends stay in the thread's registers for the write-out: in LDS they cost 3D p=2 FP64 one of
  // three workgroups per CU (150^3 brick kernel 70 -> 83 us).
  __device__ __forceinline__ void fill(const BrickArgs &br, int brick, bool full, T *v, T *halo, int nhalo,
                                       int32_t (&ends)[2]) {
    constexpr int BX = C::BX, BY = C::BY, BZ = C::BZ, LX = C::LX, LY = C::LY, LZ = C::LZ, PI = P > 1 ? P - 1 : 1;
    const int r = threadIdx.x;
    if (r >= C::NROWS) return;
    const bool yb = (r >= K1 && r < K2) || r >= K3, zb = r >= K2;
    const int rq = r - (r >= K3 ? K3 : (r >= K2 ? K2 : (r >= K1 ? K1 : 0)));
    const int ny = yb ? YB : (YI > 0 ? YI : 1), iy = rq % ny, iz = rq / ny;
    const int cy = yb ? iy : iy / PI, cz = zb ? iz : iz / PI;
    const int ly = yb ? 0 : 1 + iy - cy * PI, lz = zb ? 0 : 1 + iz - cz * PI;
    const int y = cy * P + ly, z = cz * P + lz, own = y + LY * z;
    const int64_t at = (int64_t)brick * C::NROWS + own;
    const int32_t b = br.row_base[at], hb = br.row_hbase[at];
    const uint32_t gm = full ? ~0u : br.row_gmask[at], bm = full ? ~0u : br.row_bmask[at];
    const bool edge = y == 0 || y == LY - 1 || (C::DIM == 3 && (z == 0 || z == LZ - 1));
    const int plane = (y == 0 ? 2 : 0) | (C::DIM == 3 && z == 0 ? 4 : 0);
    base[own] = b;
    first[own] = gm;
    dst[r] = edge ? halo + (int64_t)plane * nhalo + hb : v + b;
    ends[0] = br.row_hend[2 * (at - own) + own];
    ends[1] = br.row_hend[2 * (at - own) + C::NROWS + own];
    off[r] = (((cz * BY + cy) * BX * C::TILE + (lz * (P + 1) + ly) * (P + 1)) << 8) |
             (yb && cy > 0 ? kLowY : 0) | (cy < BY ? kHighY : 0) | (zb && cz > 0 ? kLowZ : 0) |
             (cz < BZ ? kHighZ : 0) | (y == 0 ? kY0 : 0) | (C::DIM == 3 && z == 0 ? kZ0 : 0);
    gmask[r] = gm;
    bmask[r] = bm;
  }
  // First DoF of the x-run (j, k) of the cell at (cx, cy, cz).
  __device__ __forceinline__ int32_t run(int cx, int cy, int cz, int j, int k) const {
    const int own = cy * P + j + C::LY * (cz * P + k);
    return base[own] + __popc(first[own] & ((1u << (cx * P)) - 1u));
  }
};

// Assembly and write-out of a brick's cells, one tile of results [z][y][x] per cell place (zero
// where there is no cell): every lattice point sums its cells' values (z, then y, then x from the
// low side: a fixed order) and is stored once.
template <typename T, class C>
__device__ __forceinline__ void brick_assemble(const T *tiles, const BrickRows<T, C> &R, const int32_t (&ends)[2],
                                               T *__restrict__ halo, int nhalo) {
  using Rows = BrickRows<T, C>;
  constexpr int P = C::P, N1 = P + 1, TS = C::TILE, BX = C::BX, BY = C::BY, LX = C::LX, NROWS = C::NROWS;
  constexpr int STEP_Y = BX * TS - P * N1, STEP_Z = BY * BX * TS - P * N1 * N1;  // to the cell before
  constexpr int DZ = C::DIM == 3 ? 1 : 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the rows' ends, all of them brick-boundary points: a row per thread
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const int r = tid < NROWS ? tid : 0, o = R.off[r];
    const int off = (o >> 8) + (side ? (BX - 1) * TS + P : 0);
    const uint32_t bm = tid < NROWS ? R.bmask[r] : 0u;
    T sum = T(0);
#pragma unroll
    for (int dz = DZ; dz >= 0; --dz)
#pragma unroll
      for (int dy = 1; dy >= 0; --dy) {
        const bool in = (o & (dy ? Rows::kLowY : Rows::kHighY)) && (o & (dz ? Rows::kLowZ : Rows::kHighZ));
        const T val = tiles[in ? off - dz * STEP_Z - dy * STEP_Y : 0];
        sum += in ? val : T(0);
      }
    const int plane = (side ? 0 : 1) | ((o & Rows::kY0) ? 2 : 0) | ((o & Rows::kZ0) ? 4 : 0);
    if ((bm >> (side ? LX - 1 : 0)) & 1u) halo[(int64_t)plane * nhalo + ends[side]] = sum;
  }
  // the points 0 < x < LX-1: lanes take whole rows, so that a lane's x is fixed, and the rows of one
  // kind sum equally many cells.  Up to four rows per lane at a time, every LDS read before the first
  // store: one by one the rows spent their time on the latency of three dependent LDS reads.
  constexpr int W = LX - 2, RPW = 64 / W, STEP = C::NW * RPW;
  static_assert(RPW >= 1, "a wavefront holds at least one row");
  const int rl = lane / W, x = 1 + lane - rl * W, cx = x / P;
  const uint32_t below = (1u << x) - 1u;
  const int xa = cx * TS + (x - cx * P), xb = (cx - 1) * TS + P;
  const bool two = x == cx * P;  // a point between two cells
  auto rows = [&](auto r0_, auto r1_, auto yb_, auto zb_) {
    constexpr int R0 = decltype(r0_)::value, R1 = decltype(r1_)::value;
    constexpr bool YB_ = decltype(yb_)::value, ZB_ = decltype(zb_)::value && DZ == 1;
    constexpr int NPASS = (R1 - R0 + STEP - 1) / STEP, CH = NPASS < 4 ? NPASS : 4;
    if constexpr (NPASS > 0) {
#pragma unroll
      for (int k0 = 0; k0 < NPASS; k0 += CH) {
        int o[CH];
        T *dst[CH];
        uint32_t gm[CH], bm[CH];
        T sum[CH];
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          const int r = R0 + wave * RPW + rl + (k0 + k) * STEP, rc = r < R1 ? r : R1 - 1;
          o[k] = R.off[rc];
          dst[k] = R.dst[rc];
          gm[k] = R.gmask[rc];
          bm[k] = r < R1 ? R.bmask[rc] : 0u;
          sum[k] = T(0);
        }
#pragma unroll
        for (int dz = ZB_ ? 1 : 0; dz >= 0; --dz)
#pragma unroll
          for (int dy = YB_ ? 1 : 0; dy >= 0; --dy) {
            const int need = (YB_ ? (dy ? Rows::kLowY : Rows::kHighY) : 0) | (ZB_ ? (dz ? Rows::kLowZ : Rows::kHighZ) : 0);
            T lo[CH], hi[CH];
#pragma unroll
            for (int k = 0; k < CH; ++k) {
              const bool in = (o[k] & need) == need;
              const int off = in ? (o[k] >> 8) - dz * STEP_Z - dy * STEP_Y : 0;
              lo[k] = tiles[in && two ? off + xb : 0];
              hi[k] = tiles[off + xa];
            }
#pragma unroll
            for (int k = 0; k < CH; ++k) {
              settle(lo[k]);
              settle(hi[k]);
              const bool in = (o[k] & need) == need;
              lo[k] = in && two ? lo[k] : T(0);
              hi[k] = in ? hi[k] : T(0);
            }
#pragma unroll
            for (int k = 0; k < CH; ++k) sum[k] += lo[k] + hi[k];
          }
#pragma unroll
        for (int k = 0; k < CH; ++k) settle(sum[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k)
          if ((bm[k] >> x) & 1u) ((GlobalT<T> *)dst[k])[__popc(gm[k] & below)] = sum[k];  // (generic: see GlobalT)
      }
    }
  };
  if (rl < RPW) {
    using std::integral_constant;
    rows(integral_constant<int, 0>{}, integral_constant<int, Rows::K1>{}, std::false_type{}, std::false_type{});
    rows(integral_constant<int, Rows::K1>{}, integral_constant<int, Rows::K2>{}, std::true_type{}, std::false_type{});
    rows(integral_constant<int, Rows::K2>{}, integral_constant<int, Rows::K3>{}, std::false_type{}, std::true_type{});
    rows(integral_constant<int, Rows::K3>{}, integral_constant<int, NROWS>{}, std::true_type{}, std::true_type{});
  }
}

template <typename T, int N1>
__device__ __forceinline__ void cells_body(const int brick, BrickArgs br, const T *__restrict__ fbuf,
                                           const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
                                           int nhalo, KTab<T, N1> tab, T scale, int parts) {
  using C = CellBrickCfg<T, N1>;
  constexpr int P = N1 - 1, NP = C::NP, HC = (N1 + 1) / 2, HF = N1 / 2, TS = C::TILE;
  constexpr int BX = C::BX, BY = C::BY, LX = C::LX, LY = C::LY;
  __shared__ T tiles[C::NW * C::CPW * TS];
  __shared__ BrickRows<T, C> rows;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c0 = br.cell_off[brick], nc = br.cell_off[brick + 1] - c0, f0 = br.face_off[brick];
  const bool full = nc == C::MAXC;
  const int wc = lane / N1, j = lane - wc * N1, c = wave * C::CPW + wc;
  const bool on = wc < C::CPW && c < nc;
  const int loc = on ? br.cell_loc[c0 + c] : 0;
  const int cface = on ? br.cell_face[c0 + c] : 0;
  int32_t ends[2] = {0, 0};
  rows.fill(br, brick, full, v, halo, nhalo, ends);
  __syncthreads();
  // the cell's place in the brick, and the lane's x-runs (j, k): the first DoF of each from its row
  const int lcx = (loc % LX) / P, lcy = (loc / LX % LY) / P, lcz = loc / (LX * LY) / P;
  int32_t run[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) run[k] = rows.run(lcx, lcy, lcz, on ? j : 0, k);
  T lo[N1], hi[N1];  // x-runs of planes k and p - k
  auto fetch = [&](int k) {
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      lo[i] = u[(int64_t)run[k] + i];
      hi[i] = 2 * k == P ? T(0) : u[(int64_t)run[P - k] + i];
    }
  };
  if (on && (parts & SBM_PART_CELLS)) fetch(0);
  T out[N1][N1];  // [z][y] at x = j
#pragma unroll
  for (int z = 0; z < N1; ++z)
#pragma unroll
    for (int y = 0; y < N1; ++y) out[z][y] = T(0);
  if (on) {
    if (parts & SBM_PART_CELLS) {
      T *const turn = tiles + wave * (C::CPW * TS) + wc * C::SC;  // plane q at q * CPW * SC
      constexpr int PL = C::CPW * C::SC;
      T ye[HC][N1], yo[HF][N1];
#pragma unroll
      for (int y = 0; y < N1; ++y) {
#pragma unroll
        for (int i = 0; i < HC; ++i) ye[i][y] = T(0);
#pragma unroll
        for (int i = 0; i < HF; ++i) yo[i][y] = T(0);
      }
      // planes k and p - k together, as their sum and difference (the z operators are
      // centrosymmetric): x sweep of the lane's run in registers, through LDS to the lane's y-line,
      // y sweep, and the plane's share of the z sweep.  The next two planes are in flight.
      auto xsweep = [&](const T (&x)[N1], T *dst) {  // a = M x, b = K x of x-run j
        const EvenOdd<T, N1> ex(x);
        EOAcc<T, N1> aa, ab;
        eo_acc<T, N1>(tab.EM, tab.OM, ex, aa.ye, aa.yo);
        eo_acc<T, N1>(tab.EK, tab.OK, ex, ab.ye, ab.yo);
        T a[N1], b[N1];
        eo_combine<T, N1>(aa.ye, aa.yo, T(1), a);
        eo_combine<T, N1>(ab.ye, ab.yo, T(1), b);
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          dst[N1 * j + i] = a[i];
          dst[PL + N1 * j + i] = b[i];
        }
      };
      auto ysweep = [&](const T *src, T (&cc)[N1], T (&e)[N1]) {  // c = M a, e = K a + M b of y-line j
        T a[N1], b[N1];
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          a[i] = src[N1 * i + j];
          b[i] = src[PL + N1 * i + j];
        }
        const EvenOdd<T, N1> ea(a), eb(b);
        EOAcc<T, N1> ac, ae;
        eo_acc<T, N1>(tab.EM, tab.OM, ea, ac.ye, ac.yo);
        eo_acc<T, N1>(tab.EK, tab.OK, ea, ae.ye, ae.yo);
        eo_acc<T, N1>(tab.EM, tab.OM, eb, ae.ye, ae.yo);
        eo_combine<T, N1>(ac.ye, ac.yo, T(1), cc);
        eo_combine<T, N1>(ae.ye, ae.yo, T(1), e);
      };
#pragma unroll
      for (int k = 0; k < HC; ++k) {
        const bool mid = 2 * k == P;
        T xe[N1], xo[N1];
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          xe[i] = mid ? lo[i] : lo[i] + hi[i];
          xo[i] = lo[i] - hi[i];
        }
        if (k + 1 < HC) fetch(k + 1);
        xsweep(xe, turn);
        if (!mid) xsweep(xo, turn + 2 * PL);
        wave_sync();
        T cc[N1], e[N1];
        ysweep(turn, cc, e);
#pragma unroll
        for (int i = 0; i < HC; ++i)
#pragma unroll
          for (int y = 0; y < N1; ++y) ye[i][y] += tab.EK[i * HC + k] * cc[y] + tab.EM[i * HC + k] * e[y];
        if (!mid) {
          ysweep(turn + 2 * PL, cc, e);
#pragma unroll
          for (int i = 0; i < HF; ++i)
#pragma unroll
            for (int y = 0; y < N1; ++y) yo[i][y] += tab.OK[i * HF + k] * cc[y] + tab.OM[i * HF + k] * e[y];
        }
        wave_sync();
      }
#pragma unroll
      for (int i = 0; i < HF; ++i)
#pragma unroll
        for (int y = 0; y < N1; ++y) {
          out[i][y] = scale * (ye[i][y] + yo[i][y]);
          out[P - i][y] = scale * (ye[i][y] - yo[i][y]);
        }
      if constexpr (N1 % 2 == 1) {
#pragma unroll
        for (int y = 0; y < N1; ++y) out[HF][y] = scale * ye[HF][y];
      }
    }
    if ((parts & SBM_PART_SBM_FACES) && cface) {
      // the rows of the cell's surrogate faces, in code order, from their (Rv, Rg) per face node
      const T *R = fbuf + (int64_t)(f0 + (cface >> 6)) * 2 * NP;
#pragma unroll
      for (int code = 0; code < 6; ++code) {
        if (!((cface >> code) & 1)) continue;
        const int a = code >> 1, s = code & 1;
        const T *Rv = R, *Rg = R + NP;
        R += 2 * NP;
        if (a == 0) {
          T dj = T(0);
#pragma unroll
          for (int i = 0; i < N1; ++i) dj = i == j ? (s ? tab.D1[i] : tab.D0[i]) : dj;
          const bool at = j == s * P;
#pragma unroll
          for (int z = 0; z < N1; ++z)
#pragma unroll
            for (int y = 0; y < N1; ++y) out[z][y] += (at ? Rv[y + N1 * z] : T(0)) + dj * Rg[y + N1 * z];
        } else {
#pragma unroll
          for (int t = 0; t < N1; ++t) {
            const T rv = Rv[j + N1 * t], rg = Rg[j + N1 * t];
#pragma unroll
            for (int i = 0; i < N1; ++i) {
              T &o = a == 1 ? out[t][i] : out[i][t];
              o += (i == s * P ? rv : T(0)) + (s ? tab.D1[i] : tab.D0[i]) * rg;
            }
          }
        }
      }
    }
  }
  // the results lie by the cell's place in the brick (a full brick's cells are in place already); a
  // missing cell's are zero
  const int place = (lcz * BY + lcy) * BX + lcx;
  if (!full) {
    __syncthreads();
    for (int i = tid; i < C::MAXC * TS; i += C::NT) tiles[i] = T(0);
    __syncthreads();
  }
  if (on) {
    T *const tile = tiles + place * TS;
#pragma unroll
    for (int z = 0; z < N1; ++z)
#pragma unroll
      for (int y = 0; y < N1; ++y) tile[(z * N1 + y) * N1 + j] = out[z][y];
  }
  __syncthreads();
  brick_assemble<T, C>(tiles, rows, ends, halo, nhalo);
}

// The rows of a cell's surrogate faces for its x-run t, in code order, from their (Rv, Rg) per face node:
// cf is the cell's entry of cell_face, F the results of the brick's first face.
template <typename T, int D, int N1>
__device__ __forceinline__ void tile_face_rows(const KTab<T, N1> &tab, const T *__restrict__ F, int cf, int t,
                                               T (&frow)[N1]) {
  constexpr int P = N1 - 1, NP = Shape<D, N1>::NP;
  const int t0 = (D == 3) ? t % N1 : t, t1 = (D == 3) ? t / N1 : 0;
  const T *Rq = F + (int64_t)(cf >> 6) * 2 * NP;
#pragma unroll
  for (int code = 0; code < 2 * D; ++code) {
    if (!((cf >> code) & 1)) continue;
    const int a = code >> 1, s = code & 1;
    const T *Rv = Rq, *Rg = Rq + NP;
    Rq += 2 * NP;
    if (a == 0) {
      const T rv = Rv[t], rg = Rg[t];
#pragma unroll
      for (int i = 0; i < N1; ++i) frow[i] += (i == s * P ? rv : T(0)) + (s ? tab.D1[i] : tab.D0[i]) * rg;
    } else {
      const int ia = a == 1 ? t0 : t1, n0 = (D == 3) ? N1 * (a == 1 ? t1 : t0) : 0;
      T da = T(0);
#pragma unroll
      for (int i = 0; i < N1; ++i) da = i == ia ? (s ? tab.D1[i] : tab.D0[i]) : da;
      const bool on = ia == s * P;
#pragma unroll
      for (int i = 0; i < N1; ++i) frow[i] += (on ? Rv[n0 + i] : T(0)) + da * Rg[n0 + i];
    }
  }
}

// ------------------------------------------------------------------------------------
// Small operators of 3D p >= 4 and of 2D: all of a brick's cell places at once, (p+1)^(d-1) threads
// each, two tiles of LDS per place; every lattice point then sums its cells' values as it is stored.
// What bounds it: the latency of its phases (row tables, gather, one pass per axis, write-out), so it
// takes the operators whose bricks are on the device all at once (kCellsMax; whole apply replayed from a
// graph, by sweeps -> now: 24^3 Q4 FP64 22.6 -> 14.4 us, FP32 20.1 -> 13.1, 2D Q2 disk of 345 unknowns 11.2
// -> 8.5; a call of its own on that disk is bound by the host's launches, 17.5 -> 16 to 18 us).
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1>
__device__ __forceinline__ void tile_body(const int brick, BrickArgs br, const T *__restrict__ fbuf,
                                          const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
                                          int nhalo, KTab<T, N1> tab, T scale, int parts) {
  using C = TileBrickCfg<T, D, N1>;
  constexpr int P = N1 - 1, NP = C::NP, NB = C::NB, BX = C::BX, BY = C::BY, BZ = C::BZ;
  constexpr int LX = C::LX, LY = C::LY;
  __shared__ T smem[C::MAXC * (C::TILE + NB)];
  __shared__ BrickRows<T, C> rows;
  __shared__ int32_t s_info[C::MAXC];  // per place: 0 without a cell, else 1 + 2 x its faces (cell_face)
  const int tid = threadIdx.x;
  const int c0 = br.cell_off[brick], nc = br.cell_off[brick + 1] - c0, f0 = br.face_off[brick];
  const int loc = tid < nc ? br.cell_loc[c0 + tid] : 0, info_ = tid < nc ? 2 * br.cell_face[c0 + tid] + 1 : 0;
  if (tid < C::MAXC) s_info[tid] = 0;
  int32_t ends[2] = {0, 0};
  rows.fill(br, brick, nc == C::MAXC, v, halo, nhalo, ends);
  __syncthreads();
  if (tid < nc) s_info[(loc / (LX * LY) / P * BY + (loc / LX % LY) / P) * BX + (loc % LX) / P] = info_;
  __syncthreads();
  const int le = tid / NP, t = tid - le * NP;
  const bool place = le < C::MAXC;
  const int info = place ? s_info[le] : 0;
  const int cx = le % BX, cy = le / BX % BY, cz = le / (BX * BY);
  const int t0 = (D == 3) ? t % N1 : t, t1 = (D == 3) ? t / N1 : 0;
  const bool work = info != 0 && (parts & SBM_PART_CELLS) != 0;
  T x[N1], out[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) {  // the pencil along the last axis
    x[k] = work ? u[(int64_t)rows.run(cx, cy, cz, (D == 3) ? t1 : k, (D == 3) ? k : 0) + t0] : T(0);
    out[k] = T(0);
  }
  // the rows of the cell's surrogate faces for x-run t, in code order, from their (Rv, Rg) per face
  // node, loaded while the pencil is under way
  T frow[N1];
#pragma unroll
  for (int i = 0; i < N1; ++i) frow[i] = T(0);
  if ((parts & SBM_PART_SBM_FACES) && (info >> 1))
    tile_face_rows<T, D, N1>(tab, fbuf + (int64_t)f0 * 2 * NP, info >> 1, t, frow);
  T *const A = smem + (place ? le : 0) * C::TILE, *const B = smem + C::MAXC * C::TILE + (place ? le : 0) * NB;
  kron_cell<T, D, N1>(tab, t, x, A, B, scale, out, work, work);
  if (place) {  // (the thread's own x-run of the tile, which it alone has read)
#pragma unroll
    for (int i = 0; i < N1; ++i) A[N1 * t + i] = out[i] + frow[i];
  }
  __syncthreads();
  brick_assemble<T, C>(smem, rows, ends, halo, nhalo);
}

// The same bricks, cells and sums, bit for bit, with PASS of the brick's cells at a time, for batches
// whose bricks fill the device several times over (tile_split): a quarter of the threads and half of the
// tiles of all places at once, so that two to three times as many bricks are on the device, the next
// cells' values under way while a pass is swept, and no work for places without a cell.
template <typename T, int N1, int SPLIT>
__device__ __forceinline__ void tile_split_body(const int brick, BrickArgs br, const T *__restrict__ fbuf,
                                                const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
                                                int nhalo, KTab<T, N1> tab, T scale) {
  using C = TileBrickCfg<T, 3, N1, SPLIT>;
  constexpr int P = N1 - 1, NP = C::NP, NB = C::NB, BX = C::BX, BY = C::BY, LX = C::LX, LY = C::LY, PASS = C::PASS;
  __shared__ T smem[C::MAXC * C::TILE + PASS * NB];
  __shared__ BrickRows<T, C> rows;
  __shared__ int32_t s_cell[C::MAXC];  // per cell: 64 x its faces (cell_face) + its place
  static_assert(C::MAXC <= 64, "a place fits six bits");
  const int tid = threadIdx.x;
  const int c0 = br.cell_off[brick], nc = br.cell_off[brick + 1] - c0;
  const T *const F = fbuf + (int64_t)br.face_off[brick] * 2 * NP;
  if (tid < nc) {
    const int loc = br.cell_loc[c0 + tid];
    s_cell[tid] = br.cell_face[c0 + tid] * 64 + (loc / (LX * LY) / P * BY + (loc / LX % LY) / P) * BX + (loc % LX) / P;
  }
  int32_t ends[2] = {0, 0};
  rows.fill(br, brick, nc == C::MAXC, v, halo, nhalo, ends);
  if (nc < C::MAXC)
    for (int i = tid; i < C::MAXC * C::TILE; i += C::NT) smem[i] = T(0);
  __syncthreads();
  const int le = tid / NP, t = tid - le * NP, t0 = t % N1, t1 = t / N1;
  auto fetch = [&](int c, int &cell, T (&x)[N1]) {
    const bool on = le < PASS && c < nc;
    cell = on ? s_cell[c] : -1;
    const int pl = on ? cell & 63 : 0;
#pragma unroll
    for (int k = 0; k < N1; ++k)
      x[k] = on ? u[(int64_t)rows.run(pl % BX, pl / BX % BY, pl / (BX * BY), t1, k) + t0] : T(0);
  };
  int cell, next = -1;
  T x[N1], y[N1] = {};
  fetch(le, cell, x);
  for (int c = 0; c < nc; c += PASS) {
    if (c + PASS < nc) fetch(c + PASS + le, next, y);
    const bool on = cell >= 0;
    T out[N1], frow[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) out[i] = frow[i] = T(0);
    if (on && (cell >> 6)) tile_face_rows<T, 3, N1>(tab, F, cell >> 6, t, frow);
    T *const A = smem + (on ? cell & 63 : 0) * C::TILE, *const B = smem + C::MAXC * C::TILE + (on ? le : 0) * NB;
    kron_cell<T, 3, N1>(tab, t, x, A, B, scale, out, on, on);
#pragma unroll
    for (int i = 0; i < N1; ++i) settle(out[i]);  // (rounded before the sum, as in tile_body)
    if (on) {
#pragma unroll
      for (int i = 0; i < N1; ++i) A[N1 * t + i] = out[i] + frow[i];
    }
    __syncthreads();
    cell = next;
#pragma unroll
    for (int i = 0; i < N1; ++i) x[i] = y[i];
  }
  brick_assemble<T, C>(smem, rows, ends, halo, nhalo);
}

template <typename T, int D, int N1, bool CELLS>
__device__ __forceinline__ void brick_body(const int blk, BrickArgs br, const T *__restrict__ fbuf,
                                           const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
                                           int nhalo, KTab<T, N1> tab, T scale, int parts) {
  if constexpr (!CELLS)
    sweeps_body<T, D, N1>(blk, br, fbuf, u, v, halo, nhalo, tab, scale, parts);
  else if constexpr (D == 3 && N1 <= 4)
    cells_body<T, N1>(blk, br, fbuf, u, v, halo, nhalo, tab, scale, parts);
  else
    tile_body<T, D, N1>(blk, br, fbuf, u, v, halo, nhalo, tab, scale, parts);
}

template <typename T, int D, int N1, bool CELLS>
__global__ __launch_bounds__((BrickCfg<T, D, N1, CELLS>::NT)) void brick_kernel(
    BrickArgs br, const T *__restrict__ fbuf, const T *__restrict__ u, T *__restrict__ v, T *__restrict__ halo,
    int nhalo, KTab<T, N1> tab, T scale, int parts) {
  brick_body<T, D, N1, CELLS>(xcd_block(), br, fbuf, u, v, halo, nhalo, tab, scale, parts);
}

// v[dof] = sum over the planes k present in the DoF's mask, in increasing k (deterministic).
// Two DoFs per thread (a block's 2 * 256 consecutive ones), so that each thread has twice the
// loads in flight (FP64 apply at 64^3 Q4: 50.2 against 51.2 us; with four 1.5 us slower).
// What bounds it: the points on x planes, each a store of one value to a cache line of v.  They are a
// sixteenth of all points at 3D p=4, and with the same stores side by side 128^3 FP64 took 45 us less when
// the pass took 110 (73 now, with nontemporal reads of the planes).  With the halo numbered for dense planes
// and stores (see build_bricks) instead of in DoF order, and the surrogate faces by one thread per point,
// 128^3 Q4 replayed: FP64 apply 404 -> 324 us, FP32 222 -> 211.  One contiguous range of it per XCD measured
// slower (128^3 FP64 381 against 357 us then).
constexpr int kHaloPerThread = 2;
template <typename T, int D, bool ONCE>
__device__ __forceinline__ void halo_reduce_body(const int blk, int n, const int32_t *__restrict__ dof,
                                                          const uint8_t *__restrict__ mask,
                                                          const T *__restrict__ halo, T *__restrict__ v) {
  const int i0 = blk * (kHaloPerThread * 256) + threadIdx.x;
  uint32_t m[kHaloPerThread];
  int dd[kHaloPerThread];
#pragma unroll
  for (int r = 0; r < kHaloPerThread; ++r) {
    const int i = i0 + r * 256;
    m[r] = i < n ? mask[i] : 0u;
    dd[r] = i < n ? dof[i] : 0;
  }
  T s[kHaloPerThread];
#pragma unroll
  for (int r = 0; r < kHaloPerThread; ++r) s[r] = T(0);
#pragma unroll
  for (int k = 0; k < (1 << D); ++k)
#pragma unroll
    for (int r = 0; r < kHaloPerThread; ++r)
      s[r] += ((m[r] >> k) & 1u) ? (ONCE ? __builtin_nontemporal_load(&halo[(int64_t)k * n + i0 + r * 256])
                                        : halo[(int64_t)k * n + i0 + r * 256]) : T(0);
#pragma unroll
  for (int r = 0; r < kHaloPerThread; ++r)
    if (i0 + r * 256 < n) v[dd[r]] = s[r];
}

template <typename T, int D, bool ONCE>
__global__ __launch_bounds__(256) void halo_reduce_kernel(int n, const int32_t *__restrict__ dof,
                                                          const uint8_t *__restrict__ mask,
                                                          const T *__restrict__ halo, T *__restrict__ v) {
  halo_reduce_body<T, D, ONCE>(blockIdx.x, n, dof, mask, halo, v);
}

// ------------------------------------------------------------------------------------
// CG surrogate-boundary faces (Alg. 3), EPB faces per workgroup, faces in brick order.
// Output per face: Rv and Rg at its NP face nodes (fbuf[f][0][t], fbuf[f][1][t]);
// brick_kernel expands them into the (p+1)^d local rows (face_row).
// Thread t of a face is face node t, then face Gauss point t.  With dn = (2s-1)/h d/dxi_a on the face
// and N the GLL -> Gauss matrix, the dn u term, N^T W N per tangential axis, is the 1D mass matrix M per
// axis on the nodes' normal derivatives: it needs no Gauss points and is swept together with
// N^T (W E u), two sweeps in all.
// What bounds it: the latency of that chain; a face's 5 kB and 10 kFLOP at 3D p=4 are small against it.
// With half of the threads for E u, two points each, and dn u taken to the Gauss points and back (four
// sweeps), kernel in us: 66^3 Q4 FP64 17.1 -> 15.5, 50^3 Q5 17.2 -> 13.6, 40^3 Q6 27.0 -> 22.0, 20^3 Q8 23.6
// -> 17.3, 36^3 Q8 49.7 -> 44.2, FP32 20^3 Q8 20.2 -> 11.4.  At Q8 the reads of the cell's 729 values from
// LDS bound it, which one thread per point does twice as often: 30^3 Q8 FP64, whose 965 workgroups fill the
// device just once, 29.3 -> 33.0.
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1, int EPB>
__device__ __forceinline__ void sbm_face_cg_body(const int blk, int n_faces, const int32_t *__restrict__ face_code,
                                                          const int32_t *__restrict__ face_runs,
                                                          const double *__restrict__ face_xi,
                                                          const T *__restrict__ u, T *__restrict__ fbuf,
                                                          KTab<T, N1> tab, KScal sc) {
  constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  __shared__ T su_all[EPB * NB];
  __shared__ T fw_all[4 * EPB * NP];  // per face: W E u, normal derivative, and both after the first sweep
  __shared__ T sN[N1 * N1], sM[N1 * N1];
  const int tid = threadIdx.x, le = tid / NP, t = tid - le * NP;
  const int f = blk * EPB + le;
  const bool act = f < n_faces;  // (the launch has EPB NP threads)
  T *su = su_all + le * NB, *fe = fw_all + le * 4 * NP, *fg = fe + NP, *re = fe + 2 * NP, *rg = fe + 3 * NP;
  // loads first: face code, the point, the cell's u (one x-run per thread)
  const int code = act ? face_code[f] : 0;
  double xp[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xp[k] = act ? face_xi[((int64_t)f * NP + t) * D + k] : 0.0;
  {
    const int64_t base = act ? face_runs[(int64_t)f * NP + t] : 0;
#pragma unroll
    for (int i = 0; i < N1; ++i) su[N1 * t + i] = act ? u[base + i] : T(0);
  }
  for (int i = tid; i < N1 * N1; i += EPB * NP) {
    sN[i] = tab.N[i];
    sM[i] = tab.M[i];
  }
  T l[D][N1];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    double lk[N1];
    lagrange_at<N1>(tab.z, tab.cinv, xp[k], lk);
#pragma unroll
    for (int j = 0; j < N1; ++j) l[k][j] = T(lk[j]);
  }
  __syncthreads();
  const FaceAxes<D, N1> fa(code);
  const int jb = (D == 3) ? t % N1 : t, jc = (D == 3) ? t / N1 : 0;
  const T h = T(sc.h), sig = T(sc.sigma_gamma), sh = (fa.s ? T(1) : T(-1)) / h;
  {
    T g = 0;
    const int node_off = jb * fa.Sb + jc * fa.Sc;
#pragma unroll
    for (int ia = 0; ia < N1; ++ia) g += (fa.s ? tab.D1[ia] : tab.D0[ia]) * su[ia * fa.Sa + node_off];
    fg[t] = g;
  }
  {
    T e = 0;
    if constexpr (D == 3) {
#pragma unroll
      for (int i2 = 0; i2 < N1; ++i2) {
        T r = 0;
#pragma unroll
        for (int i1 = 0; i1 < N1; ++i1) {
          T q = 0;
#pragma unroll
          for (int i0 = 0; i0 < N1; ++i0) q += l[0][i0] * su[i0 + N1 * i1 + NP * i2];
          r += l[1][i1] * q;
        }
        T l2 = 0;
#pragma unroll
        for (int j = 0; j < N1; ++j) l2 = (j == i2) ? l[2][j] : l2;
        e += l2 * r;
      }
    } else {
#pragma unroll
      for (int i1 = 0; i1 < N1; ++i1) {
        T q = 0;
#pragma unroll
        for (int i0 = 0; i0 < N1; ++i0) q += l[0][i0] * su[i0 + N1 * i1];
        e += l[1][i1] * q;
      }
    }
    fe[t] = ((D == 3) ? h * h * tab.w[t % N1] * tab.w[t / N1] : h * tab.w[t]) * e;
  }
  __syncthreads();
  T ae = 0, ag = 0;
  if constexpr (D == 3) {
    T r1 = 0, r2 = 0;
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      r1 += sN[k * N1 + jc] * fe[jb + N1 * k];
      r2 += sM[k * N1 + jc] * fg[jb + N1 * k];
    }
    re[t] = r1;
    rg[t] = r2;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      ae += sN[k * N1 + jb] * re[k + N1 * jc];
      ag += sM[k * N1 + jb] * rg[k + N1 * jc];
    }
  } else {
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      ae += sN[k * N1 + t] * fe[k];
      ag += sM[k * N1 + t] * fg[k];
    }
  }
  if (act) {
    fbuf[(int64_t)f * 2 * NP + t] = sig * ae - ((D == 3) ? h * h : h) * sh * ag;  // tested against v
    fbuf[(int64_t)f * 2 * NP + NP + t] = -sh * ae;  // tested against the reference derivative along a
  }
}

// (at least 4 waves per SIMD: keeps the scheduler from holding the whole tile in registers)
template <typename T, int D, int N1, int EPB>
__global__ __launch_bounds__(256, 4) void sbm_face_cg_kernel(int n_faces, const int32_t *__restrict__ face_code,
                                                          const int32_t *__restrict__ face_runs,
                                                          const double *__restrict__ face_xi,
                                                          const T *__restrict__ u, T *__restrict__ fbuf,
                                                          KTab<T, N1> tab, KScal sc) {
  sbm_face_cg_body<T, D, N1, EPB>(xcd_block(), n_faces, face_code, face_runs, face_xi, u, fbuf, tab, sc);
}

// DG surrogate-boundary faces: one entity = one face.  Output per face: Rv and Rg at its NP
// face nodes (fbuf[f][0][t], fbuf[f][1][t]); the DG cell kernels add the face's rows into the
// cell's block in face order, so the apply has no atomics and is bitwise reproducible.
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1, int EPB>
__device__ __forceinline__ void sbm_face_body(const int blk, int n_faces, const int32_t *__restrict__ face_cell,
                                                       const int32_t *__restrict__ face_code,
                                                       const double *__restrict__ face_xi, const T *__restrict__ u,
                                                       T *__restrict__ fbuf, KTab<T, N1> tab, KScal sc) {
  constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  __shared__ T su_all[EPB * NB];
  __shared__ T f_all[4 * EPB * NP];
  const int le = threadIdx.x / NP, t = threadIdx.x - le * NP;
  const int f = blk * EPB + le;
  const bool act = f < n_faces;
  T *su = su_all + le * NB;
  T *f1 = f_all + le * NP, *f2 = f1 + EPB * NP, *f3 = f2 + EPB * NP, *f4 = f3 + EPB * NP;
  double xp[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xp[k] = act ? face_xi[((int64_t)f * NP + t) * D + k] : 0.0;
  const FaceAxes<D, N1> fa(act ? face_code[f] : 0);
  const int64_t base = (int64_t)(act ? face_cell[f] : 0) * NB + N1 * t;
  if (act) {
#pragma unroll
    for (int i = 0; i < N1; ++i) su[N1 * t + i] = u[base + i];
  }
  __syncthreads();
  T Rv, Rg;
  sbm_face_eval<T, D, N1>(tab, sc, t, act, fa, xp, su, f1, f2, f3, f4, Rv, Rg);
  if (act) {
    fbuf[(int64_t)f * 2 * NP + t] = Rv;
    fbuf[(int64_t)f * 2 * NP + NP + t] = Rg;
  }
}

template <typename T, int D, int N1, int EPB>
__global__ __launch_bounds__(256) void sbm_face_kernel(int n_faces, const int32_t *__restrict__ face_cell,
                                                       const int32_t *__restrict__ face_code,
                                                       const double *__restrict__ face_xi, const T *__restrict__ u,
                                                       T *__restrict__ fbuf, KTab<T, N1> tab, KScal sc) {
  sbm_face_body<T, D, N1, EPB>(xcd_block(), n_faces, face_cell, face_code, face_xi, u, fbuf, tab, sc);
}

// DG surrogate-boundary faces in 3D with (p+1)^3 threads per face: thread (t, i2) takes face
// point t and slab i2 of the cell.  The cell's values are loaded one per thread; E u at each
// shifted point is split over the slabs (each thread one slab's (p+1)^2 terms) and the slab
// sums are added in slab order, as in sbm_face_eval; the face-node phases (normal
// derivative, Gauss interpolation, integration) run in every slab with identical results;
// slab 0 stores the face's (Rv, Rg) as sbm_face_kernel does.  For p <= 5 ((p+1)^3 <= 256).
template <typename T, int N1, int EPB>
__device__ __forceinline__ void sbm_face_slab_body(const int blk, int n_faces, const int32_t *__restrict__ face_cell,
                                                            const int32_t *__restrict__ face_code,
                                                            const double *__restrict__ face_xi,
                                                            const T *__restrict__ u, T *__restrict__ fbuf,
                                                            KTab<T, N1> tab, KScal sc) {
  constexpr int D = 3, NP = N1 * N1, NB = NP * N1;
  __shared__ T su_all[EPB * NB];
  __shared__ T sp_all[EPB * NB];  // slab partial sums of E u
  __shared__ T f_all[4 * EPB * NP];
  const int le = threadIdx.x / NB, r = threadIdx.x - le * NB;
  const int t = r % NP, i2 = r / NP;
  const int f = blk * EPB + le;
  const bool act = f < n_faces;
  T *su = su_all + le * NB, *sp = sp_all + le * NB;
  T *f1 = f_all + le * NP, *f2 = f1 + EPB * NP, *f3 = f2 + EPB * NP, *f4 = f3 + EPB * NP;
  double xp[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xp[k] = act ? face_xi[((int64_t)f * NP + t) * D + k] : 0.0;
  const FaceAxes<D, N1> fa(act ? face_code[f] : 0);
  if (act) su[r] = u[(int64_t)face_cell[f] * NB + r];
  __syncthreads();
  const T h = T(sc.h), sig = T(sc.sigma_gamma);
  const T sh = (fa.s ? T(1) : T(-1)) / h;
  const int jb = t % N1, jc = t / N1;
  const int node_off = jb * fa.Sb + jc * fa.Sc;
  {
    T g = 0;
#pragma unroll
    for (int ia = 0; ia < N1; ++ia) g += (fa.s ? tab.D1[ia] : tab.D0[ia]) * su[ia * fa.Sa + node_off];
    f1[t] = g;
    f2[t] = g;
  }
  __syncthreads();
  T dn, dn2;
  face_interpolate<T, D, N1>(tab, t, f1, f2, f3, f4, dn, dn2);
  dn *= sh;
  // slab i2 of E u at point t
  T part = 0;
  if (act) {
    double l[D][N1];
#pragma unroll
    for (int k = 0; k < D; ++k) lagrange_at<N1>(tab.z, tab.cinv, xp[k], l[k]);
    T s1 = 0;
#pragma unroll
    for (int i1 = 0; i1 < N1; ++i1) {
      T s0 = 0;
#pragma unroll
      for (int i0 = 0; i0 < N1; ++i0) s0 += T(l[0][i0]) * su[i0 + N1 * i1 + NP * i2];
      s1 += T(l[1][i1]) * s0;
    }
    T l2 = 0;
#pragma unroll
    for (int j = 0; j < N1; ++j) l2 = (j == i2) ? T(l[2][j]) : l2;
    part = l2 * s1;
  }
  sp[i2 * NP + t] = part;
  __syncthreads();  // slab sums written; face_interpolate's reads of f3/f4 are done
  T eu = 0;
#pragma unroll
  for (int j = 0; j < N1; ++j) eu += sp[j * NP + t];
  const T om = act ? h * h * tab.w[t % N1] * tab.w[t / N1] : T(0);
  f3[t] = om * (sig * eu - dn);  // tested against v
  f4[t] = -om * eu * sh;         // tested against the reference derivative along a
  __syncthreads();
  T Rv, Rg;
  face_integrate<T, D, N1>(tab, t, f1, f2, f3, f4, Rv, Rg);
  if (act && i2 == 0) {
    fbuf[(int64_t)f * 2 * NP + t] = Rv;
    fbuf[(int64_t)f * 2 * NP + NP + t] = Rg;
  }
}

template <typename T, int N1, int EPB>
__global__ __launch_bounds__(256) void sbm_face_slab_kernel(int n_faces, const int32_t *__restrict__ face_cell,
                                                            const int32_t *__restrict__ face_code,
                                                            const double *__restrict__ face_xi,
                                                            const T *__restrict__ u, T *__restrict__ fbuf,
                                                            KTab<T, N1> tab, KScal sc) {
  sbm_face_slab_body<T, N1, EPB>(xcd_block(), n_faces, face_cell, face_code, face_xi, u, fbuf, tab, sc);
}

// ------------------------------------------------------------------------------------
// DG cell kernel: Laplace cell term + SIPG terms of the cell's interior faces, computed
// from the cell's side only (each interior face is evaluated twice, once per cell), so
// every cell writes only its own block: no atomics, deterministic.
// For the face (a, s) of K with neighbour N and outward normal n_K = (2s-1) e_a:
//   [u]_K = u_K - u_N,  {du/dn_K} = (du_K/dn_K + du_N/dn_K)/2,
//   K's rows += int (sigma_F [u]_K - {du/dn_K}) v - 1/2 [u]_K dv/dn_K   (Alg. 2, per side)
//
// The face integral is a tensor product too: its Gauss rule is the one of the cell, so the
// interpolation to the face's points and its transpose multiply out to the 1D mass matrix M
// along each tangential axis, and the face term of axis a is M x M x (an operator along a that
// acts on the cell's line and the neighbours' adjoining lines).  With W_a that operator plus
// the stiffness matrix K,
//   v_K = h^(d-2) sum_a (M along the other axes) W_a (u_K, u_left, u_right),
// and no face values are ever interpolated or integrated.
//
// Layout: NP = (p+1)^(d-1) threads per cell, one line of p+1 nodes each; every thread forms its
// line of all d axes straight from global memory (its own and the two neighbours' values: each
// needs the whole adjoining line for the normal derivative), then
//   3D: v = M_z (M_y X + M_x Y) + M_y M_x Z,  2D: v = M_y X + M_x Y   (X = W_x u, ...),
// one LDS tile per term, the lines of every tile padded to an odd length.
// What bounds it: instruction issue and the latency of its loads.  At 80^3 Q3 FP64 (40,308
// cells) evaluating the faces one by one (traces, Gauss interpolation, integration and the rows
// of six faces) took 61.1 us and 22.2 M vector instructions of the wavefronts, 70 % of the issue
// slots; this form takes 19.0 us and 4.1 M (50 %), 2.4 TB/s of the 46 MB it must move.  32^3 Q5
// FP32 (2,008 cells): 10.9 -> 6.1 us.
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1>
struct DgCell {
  static constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  static constexpr int PITCH = N1 | 1;       // odd: lines along x fall on different LDS banks
  static constexpr int TILE = NP * PITCH;    // one term of one cell
  static constexpr bool IN_WAVE = 64 % NP == 0;  // a cell's threads share a wavefront: no barriers
  // cells per workgroup: up to 256 threads and about 40 KB
  static constexpr int full() {
    int e = 256 / NP;
    if (e < 1) e = 1;
    while (e > 1 && e * D * TILE * (int)sizeof(T) > 40000) --e;
    return e;
  }
  // few cells: one wavefront (at least one cell)
  static constexpr int few() { return 64 / NP < 1 ? 1 : (64 / NP < full() ? 64 / NP : full()); }
  __device__ static __forceinline__ void sync() {
    if constexpr (IN_WAVE) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  }
};

// y = A x for a centrosymmetric 1D matrix given by its even/odd parts.
template <typename T, int N1>
__device__ __forceinline__ void eo_mul(const T *E, const T *O, const T (&x)[N1], T (&y)[N1]) {
  const EvenOdd<T, N1> ex(x);
  EOAcc<T, N1> a;
  eo_acc<T, N1>(E, O, ex, a.ye, a.yo);
  eo_combine<T, N1>(a.ye, a.yo, T(1), y);
}

// w = W (x; l, r): the stiffness matrix on the cell's line x plus the SIPG terms of its two end
// faces against the neighbours' lines l and r (scaled by 1/h^(d-2); sh = sigma_F h).
template <typename T, int N1>
__device__ __forceinline__ void dg_line(const KTab<T, N1> &tab, T sh, const T (&x)[N1], bool has_l, const T (&l)[N1],
                                        bool has_r, const T (&r)[N1], T (&w)[N1]) {
  constexpr int P = N1 - 1;
  eo_mul<T, N1>(tab.EK, tab.OK, x, w);
  T k0 = 0, k1 = 0, n0 = 0, n1 = 0;  // own and neighbours' reference derivatives at both ends
#pragma unroll
  for (int i = 0; i < N1; ++i) {
    k0 += tab.D0[i] * x[i];
    k1 += tab.D1[i] * x[i];
    n0 += tab.D1[i] * l[i];
    n1 += tab.D0[i] * r[i];
  }
  const T j0 = x[0] - l[P], j1 = x[P] - r[0];  // jumps [u]_K
  const T c0 = has_l ? sh * j0 + T(0.5) * (k0 + n0) : T(0), g0 = has_l ? T(0.5) * j0 : T(0);
  const T c1 = has_r ? sh * j1 - T(0.5) * (k1 + n1) : T(0), g1 = has_r ? T(-0.5) * j1 : T(0);
#pragma unroll
  for (int i = 0; i < N1; ++i) w[i] += tab.D0[i] * g0 + tab.D1[i] * g1;
  w[0] += c0;
  w[P] += c1;
}

template <typename T, int D, int N1, int EPB>
__device__ __forceinline__ void dg_cell_body(const int blk, int n_cells, const int32_t *__restrict__ nbr,
                                                      const T *__restrict__ u, const T *__restrict__ fbuf,
                                                      T *__restrict__ v, KTab<T, N1> tab, KScal sc, T scale,
                                                      int parts) {
  using C = DgCell<T, D, N1>;
  constexpr int NP = C::NP, NB = C::NB, P = N1 - 1, LP = C::PITCH;
  __shared__ T tiles[EPB * D * C::TILE];
  const int le = threadIdx.x / NP, t = threadIdx.x - le * NP;
  const int cell = blk * EPB + le;
  const bool act = cell < n_cells;
  const bool use_int = (parts & SBM_PART_CELLS) != 0, use_sbm = (parts & SBM_PART_SBM_FACES) != 0;
  T *A = tiles + le * D * C::TILE, *B = A + C::TILE, *Z = B + (D == 3 ? C::TILE : 0);
  const T sh = T(sc.sigma_f * sc.h);
  int nbs[2 * D];
#pragma unroll
  for (int k = 0; k < 2 * D; ++k) nbs[k] = act ? nbr[(int64_t)cell * 2 * D + k] : -1;
  // line t along axis a: node i at g0 + i * gs in the cell's block, at s0 + i * ss in its tiles
  const int t0 = (D == 3) ? t % N1 : t, t1 = (D == 3) ? t / N1 : 0;
  const int g0[3] = {N1 * t, (D == 3) ? t0 + NP * t1 : t, t}, gs[3] = {1, N1, NP};
  const int s0[3] = {LP * t, (D == 3) ? t0 + LP * N1 * t1 : t, t0 + LP * t1}, ss[3] = {1, LP, LP * N1};
  T out[N1];
#pragma unroll
  for (int i = 0; i < N1; ++i) out[i] = T(0);
  // surrogate faces (-2 - nbr): the rows of their (Rv, Rg), in face order.  The thread holds the
  // line along the last axis, so a face of another axis meets it in one node line of the face.
  constexpr int aL = D - 1;
  // Few cells: every load ahead of the first use (192 registers at most), the faces' also where there is
  // none.  Axis after axis and face after face they took 3D Q3, 7 cells, FP64, 7.9 us on the device against
  // 6.5 (replayed apply), 3D Q2, 373 cells, 7.7 against 6.2.
  constexpr bool AHEAD = EPB < C::full() && ((3 * D + 4 * (D - 1)) * N1 + 4) * sizeof(T) <= 768;
  T rv[2 * D][N1], rg[2 * D][N1];
  if constexpr (AHEAD) {
#pragma unroll
    for (int code = 0; code < 2 * D; ++code) {
      const bool has = use_sbm && nbs[code] < -1;
      const T *Rv = has ? fbuf + (int64_t)(-2 - nbs[code]) * 2 * NP : u;  // (u has a cell's values at least)
      const int a = code >> 1, n0 = a == aL ? t : (D == 3 ? (a == 0 ? t1 : t0) : 0);
#pragma unroll
      for (int i = 0; i < (a == aL ? 1 : N1); ++i) {
        rv[code][i] = Rv[n0 + (D == 3 ? N1 * i : i)];
        rg[code][i] = Rv[NP + n0 + (D == 3 ? N1 * i : i)];
      }
    }
  }
  if (use_int) {
    const int64_t own = (int64_t)(act ? cell : 0) * NB;
    T xs[AHEAD ? D : 1][N1], ls[AHEAD ? D : 1][N1], rs[AHEAD ? D : 1][N1];
    if constexpr (AHEAD) {
#pragma unroll
      for (int a = 0; a < D; ++a)
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          xs[a][i] = u[own + g0[a] + i * gs[a]];
          ls[a][i] = u[(nbs[2 * a] >= 0 ? (int64_t)nbs[2 * a] * NB : own) + g0[a] + i * gs[a]];
          rs[a][i] = u[(nbs[2 * a + 1] >= 0 ? (int64_t)nbs[2 * a + 1] * NB : own) + g0[a] + i * gs[a]];
        }
#pragma unroll
      for (int a = 0; a < D; ++a)
#pragma unroll
        for (int i = 0; i < N1; ++i) {
          settle(xs[a][i]);
          settle(ls[a][i]);
          settle(rs[a][i]);
        }
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const bool has_l = nbs[2 * a] >= 0, has_r = nbs[2 * a + 1] >= 0;
      // (a missing neighbour reads the cell itself; what is made of it is dropped)
      const T *up = u + own + g0[a];
      const T *lp = u + (has_l ? (int64_t)nbs[2 * a] * NB : own) + g0[a];
      const T *rp = u + (has_r ? (int64_t)nbs[2 * a + 1] * NB : own) + g0[a];
      T x[N1], l[N1], r[N1], w[N1];
#pragma unroll
      for (int i = 0; i < N1; ++i) {
        x[i] = AHEAD ? xs[AHEAD ? a : 0][i] : up[i * gs[a]];
        l[i] = AHEAD ? ls[AHEAD ? a : 0][i] : lp[i * gs[a]];
        r[i] = AHEAD ? rs[AHEAD ? a : 0][i] : rp[i * gs[a]];
      }
      dg_line<T, N1>(tab, sh, x, has_l, l, has_r, r, w);
      T *dst = (a == 0 ? A : (a == 1 ? B : Z)) + s0[a];
#pragma unroll
      for (int i = 0; i < N1; ++i) dst[i * ss[a]] = w[i];
    }
    C::sync();
    auto sweep = [&](T *tile, int a) {  // the tile's line t along axis a times M, in place
      T x[N1], y[N1];
#pragma unroll
      for (int i = 0; i < N1; ++i) x[i] = tile[s0[a] + i * ss[a]];
      eo_mul<T, N1>(tab.EM, tab.OM, x, y);
#pragma unroll
      for (int i = 0; i < N1; ++i) tile[s0[a] + i * ss[a]] = y[i];
    };
    if constexpr (D == 3) {
      sweep(A, 1);
      sweep(B, 0);
      sweep(Z, 0);
      C::sync();
      sweep(Z, 1);
      T x[N1], y[N1];
#pragma unroll
      for (int i = 0; i < N1; ++i) x[i] = A[s0[2] + i * ss[2]] + B[s0[2] + i * ss[2]];
      eo_mul<T, N1>(tab.EM, tab.OM, x, y);
      C::sync();
#pragma unroll
      for (int i = 0; i < N1; ++i) out[i] = scale * (y[i] + Z[s0[2] + i * ss[2]]);
    } else {
      sweep(B, 0);
      T x[N1], y[N1];
#pragma unroll
      for (int i = 0; i < N1; ++i) x[i] = A[s0[1] + i * ss[1]];
      eo_mul<T, N1>(tab.EM, tab.OM, x, y);
      C::sync();
#pragma unroll
      for (int i = 0; i < N1; ++i) out[i] = scale * (y[i] + B[s0[1] + i * ss[1]]);
    }
  }
  if (!act) return;
  if (use_sbm) {
#pragma unroll
    for (int code = 0; code < 2 * D; ++code) {
      if (nbs[code] >= -1) continue;
      const int a = code >> 1, s = code & 1;
      const T *Rv = fbuf + (int64_t)(-2 - nbs[code]) * 2 * NP, *Rg = Rv + NP;
      if (a == aL) {
        const T rv0 = AHEAD ? rv[code][0] : Rv[t], rg0 = AHEAD ? rg[code][0] : Rg[t];
#pragma unroll
        for (int i = 0; i < N1; ++i) out[i] += (i == s * P ? rv0 : T(0)) + (s ? tab.D1[i] : tab.D0[i]) * rg0;
      } else {
        const int ia = a == 0 ? t0 : t1;  // the line's place along the face's normal
        const int n0 = (D == 3) ? (a == 0 ? t1 : t0) : 0;
        T dia = T(0);
#pragma unroll
        for (int i = 0; i < N1; ++i) dia = i == ia ? (s ? tab.D1[i] : tab.D0[i]) : dia;
        if constexpr (AHEAD) {
#pragma unroll
          for (int i = 0; i < N1; ++i) out[i] += (ia == s * P ? rv[code][i] : T(0)) + dia * rg[code][i];
        } else {
#pragma unroll
          for (int i = 0; i < N1; ++i) {
            const int node = (D == 3) ? n0 + N1 * i : i;
            out[i] += (ia == s * P ? Rv[node] : T(0)) + dia * Rg[node];
          }
        }
      }
    }
  }
  T *vp = v + (int64_t)cell * NB + g0[aL];
#pragma unroll
  for (int i = 0; i < N1; ++i) vp[i * gs[aL]] = out[i];
}

template <typename T, int D, int N1, int EPB>
__global__ __launch_bounds__(256) void dg_cell_kernel(int n_cells, const int32_t *__restrict__ nbr,
                                                      const T *__restrict__ u, const T *__restrict__ fbuf,
                                                      T *__restrict__ v, KTab<T, N1> tab, KScal sc, T scale,
                                                      int parts) {
  dg_cell_body<T, D, N1, EPB>(xcd_block(), n_cells, nbr, u, fbuf, v, tab, sc, scale, parts);
}

template <typename T, int N1>
KTab<T, N1> make_ktab(const Rules1D &r) {
  KTab<T, N1> k;
  constexpr int HC = (N1 + 1) / 2, HF = N1 / 2, P = N1 - 1;
  const std::vector<double> *mats[2] = {&r.M, &r.K};
  T *E[2] = {k.EM, k.EK}, *O[2] = {k.OM, k.OK};
  for (int m = 0; m < 2; ++m) {
    const std::vector<double> &A = *mats[m];
    for (int i = 0; i < HC; ++i)
      for (int c = 0; c < HC; ++c)
        E[m][i * HC + c] = T(c < HF ? 0.5 * (A[i * N1 + c] + A[i * N1 + (P - c)]) : A[i * N1 + c]);
    for (int i = 0; i < HF; ++i)
      for (int c = 0; c < HF; ++c) O[m][i * HF + c] = T(0.5 * (A[i * N1 + c] - A[i * N1 + (P - c)]));
  }
  for (int i = 0; i < N1 * N1; ++i) {
    k.M[i] = T(r.M[i]);
    k.K[i] = T(r.K[i]);
    k.N[i] = T(r.N[i]);
  }
  for (int j = 0; j < N1; ++j) {
    k.D0[j] = T(r.D0[j]);
    k.D1[j] = T(r.D1[j]);
    k.w[j] = T(r.w[j]);
    k.z[j] = r.z[j];
    k.cinv[j] = r.cinv[j];
  }
  return k;
}

template <typename T, int D, int N1>
hipError_t apply_impl(const sbm_ctx *c, const T *u, T *v, int parts, hipStream_t s, const Scratch &scr) {
  constexpr int NP = Shape<D, N1>::NP;
  const KTab<T, N1> tab = make_ktab<T, N1>(c->rules);
  const KScal sc{c->h, c->sigma_gamma, c->sigma_f};
  const T scale = T(D == 3 ? c->h : 1.0);
  const int nc = (int)c->n_cells, nf = (int)c->n_sbm;
  if (c->disc == SBM_CG) {
    if (c->n_bricks > 0 && (parts & (SBM_PART_CELLS | SBM_PART_SBM_FACES))) {
      const BrickArgs br{c->d_brick_cell_off, c->d_brick_runs, c->d_brick_cell_loc, c->d_brick_face_off,
                         c->d_brick_face_loc, c->d_face_code,  c->d_brick_cell_face, c->d_row_base,       c->d_row_gmask,
                         c->d_row_bmask,      c->d_row_hbase,     c->d_row_hend};
      T *halo = (T *)scr.halo;
      T *fbuf = (T *)scr.fbuf;
      if (nf > 0 && (parts & SBM_PART_SBM_FACES) && !(parts & SBM_PART_REUSE_FACES)) {
        // (the one-thread-per-(point, slab) layout of the DG faces measured 21.7 against 11.6 us here
        // at 3D p = 4)
        constexpr int EF = epb<T, D, N1, 2, 0>();
        hipLaunchKernelGGL((sbm_face_cg_kernel<T, D, N1, EF>), dim3((nf + EF - 1) / EF), dim3(EF * NP), 0, s, nf,
                           c->d_face_code, c->d_face_runs, c->d_face_xi, u, fbuf, tab, sc);
      }
      const int nh = (int)c->n_halo_dofs;
      auto bricks = [&](auto by_cells) {
        constexpr bool CELLS = decltype(by_cells)::value;
        hipLaunchKernelGGL((brick_kernel<T, D, N1, CELLS>), dim3((unsigned)c->n_bricks),
                           dim3(BrickCfg<T, D, N1, CELLS>::NT), 0, s, br, (const T *)fbuf, u, v, halo, nh, tab, scale,
                           parts);
      };
      if (c->by_cells) bricks(std::true_type{});
      if constexpr (has_sweeps<D, N1>())
        if (!c->by_cells) bricks(std::false_type{});
      if (nh > 0 && !(parts & SBM_PART_NO_ASSEMBLY)) {
        constexpr int HB = kHaloPerThread * 256;  // DoFs per block
        auto reduce = [&](auto once) {
          hipLaunchKernelGGL((halo_reduce_kernel<T, D, decltype(once)::value>), dim3((nh + HB - 1) / HB), dim3(256), 0,
                             s, nh, c->d_halo_dof, (const uint8_t *)c->d_halo_mask, (const T *)halo, v);
        };
        // nontemporal reads of the planes once an apply's data is several times the 256 MB cache, in FP64:
        // 128^3 Q4 (8.1 M points) 340 -> 323 us, 112^3 (5.4 M) 220 -> 216 us; on 64^3 (1.0 M) they cost a
        // solver's repeated applies 47.9 -> 51.5 us, 80^3 (2.0 M) 76 -> 83 us; FP32 64^3 39.5 -> 40.9 us
        if (sizeof(T) == 8 && nh >= 1 << 22)
          reduce(std::true_type{});
        else
          reduce(std::false_type{});
      }
    }
  } else {
    // surrogate faces first (their (Rv, Rg) go to fbuf), then the cell kernel writes every
    // cell's block once: cell term, interior faces and the surrogate faces' rows in face order
    T *fbuf = (T *)scr.fbuf;
    if (nf > 0 && (parts & SBM_PART_SBM_FACES) && !(parts & SBM_PART_REUSE_FACES)) {
      if constexpr (D == 3 && Shape<D, N1>::NB <= 256) {
        constexpr int NB = Shape<D, N1>::NB, E = 256 / NB, E1 = (64 / NB < 1) ? 1 : 64 / NB;
        if ((nf + E - 1) / E >= two_per_cu())
          hipLaunchKernelGGL((sbm_face_slab_kernel<T, N1, E>), dim3((nf + E - 1) / E), dim3(E * NB), 0, s, nf,
                             c->d_face_cell, c->d_face_code, c->d_face_xi, u, fbuf, tab, sc);
        else
          hipLaunchKernelGGL((sbm_face_slab_kernel<T, N1, E1>), dim3((nf + E1 - 1) / E1), dim3(E1 * NB), 0, s,
                             nf, c->d_face_cell, c->d_face_code, c->d_face_xi, u, fbuf, tab, sc);
      } else {
        constexpr int E = epb<T, D, N1, 1, 0>(), E1 = epb_one_wave<T, D, N1, 1>();
        if ((nf + E - 1) / E >= two_per_cu())
          hipLaunchKernelGGL((sbm_face_kernel<T, D, N1, E>), dim3((nf + E - 1) / E), dim3(E * NP), 0, s, nf,
                             c->d_face_cell, c->d_face_code, c->d_face_xi, u, fbuf, tab, sc);
        else
          hipLaunchKernelGGL((sbm_face_kernel<T, D, N1, E1>), dim3((nf + E1 - 1) / E1), dim3(E1 * NP), 0, s, nf,
                             c->d_face_cell, c->d_face_code, c->d_face_xi, u, fbuf, tab, sc);
      }
    }
    // entities per workgroup: as many as fit, unless that leaves fewer than two workgroups
    // per compute unit; then one wavefront's worth
    if (nc > 0 && (parts & (SBM_PART_CELLS | SBM_PART_SBM_FACES))) {
      using DC = DgCell<T, D, N1>;
      constexpr int E = DC::full(), E1 = DC::few();
      if ((nc + E - 1) / E >= two_per_cu())
        hipLaunchKernelGGL((dg_cell_kernel<T, D, N1, E>), dim3((nc + E - 1) / E), dim3(E * NP), 0, s, nc, c->d_nbr, u,
                           (const T *)fbuf, v, tab, sc, scale, parts);
      else
        hipLaunchKernelGGL((dg_cell_kernel<T, D, N1, E1>), dim3((nc + E1 - 1) / E1), dim3(E1 * NP), 0, s, nc, c->d_nbr,
                           u, (const T *)fbuf, v, tab, sc, scale, parts);
    }
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Batched applies: the applies of several operators that share a kernel instantiation
// (discretisation, dimension, degree, precision) run as one launch per stage over all of
// them (surrogate faces, cells or bricks, brick-boundary sums).  Workgroup g of a stage finds
// its item through blk_item[g] and runs the body of the single apply with that item's arrays
// and its block index inside the item, so every item's result is bitwise the one of its own
// apply.  The DG stages use the many-entities-per-workgroup variants (a batch fills the device).
// ------------------------------------------------------------------------------------

template <typename T, int D, int N1>
struct BatchShape {
  static constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB;
  static constexpr int EF = epb<T, D, N1, 2, 0>();  // CG faces per workgroup (as the single apply)
  // DG faces: the slab layout in 3D where a cell fits one workgroup, else one group per face
  static constexpr bool SLAB = D == 3 && NB <= 256;
  static constexpr int EFD = SLAB ? 256 / NB : epb<T, D, N1, 1, 0>();
  static constexpr int TFD = SLAB ? EFD * NB : EFD * NP;
  // DG cells per workgroup, as for the single apply: few where full ones leave the device without two each
  static constexpr int EC = DgCell<T, D, N1>::full(), EC1 = DgCell<T, D, N1>::few();
};

template <typename T, int D, int N1>
__global__ __launch_bounds__((TileBrickCfg<T, D, N1, tile_split<D, N1>()>::NT)) void brick_split_batch_kernel(
    const BatchItem *__restrict__ items, const int32_t *__restrict__ blk_item, KTab<T, N1> tab) {
  const int g = xcd_block();
  const BatchItem it = batch_item(items, blk_item[g]);
  tile_split_body<T, N1, tile_split<D, N1>()>(g - it.blk0[3], it.br, (const T *)it.fbuf, (const T *)it.u, (T *)it.v,
                                              (T *)it.halo, it.nh, tab, T(it.sc.h));
}

template <typename T, int D, int N1, bool CELLS>
__global__ __launch_bounds__((BrickCfg<T, D, N1, CELLS>::NT)) void brick_batch_kernel(const BatchItem *__restrict__ items,
                                                                              const int32_t *__restrict__ blk_item,
                                                                              KTab<T, N1> tab) {
  const int g = xcd_block();
  BatchItem it = batch_item(items, blk_item[g]);
  // The sweeps of the high degrees fill the scalar registers with the 1D tables, and what does not fit is
  // kept in lanes of vector registers: the item's pointers go to vector registers instead (3D Q6 FP64:
  // 978 reads of such lanes of 2,967 instructions, 158 of 2,207 now).  By cells they cost 3D Q8 a resident
  // workgroup, and the low degrees have no such spill.  With the pointers marked global, a prepared batch of
  // one ball (disk), us, flat and scalar / now: 40^3 Q6 FP64 90.5 / 80.0, 50^3 Q5 85.1 / 80.1, 66^3 Q4 83.7 /
  // 78.5, 30^3 Q8 113.5 / 110.1 and FP32 66.3 / 61.6, 260^2 Q6 33.7 / 30.0
  if constexpr (!CELLS && sizeof(T) * N1 * N1 >= 256) {
    auto vec = [](auto *&p) {
      using P = std::remove_pointer_t<std::remove_reference_t<decltype(p)>>;
      uintptr_t a = (uintptr_t)p;
      settle(a);
      p = (P *)(GlobalT<P> *)a;
    };
    vec(it.u);
    vec(it.v);
    vec(it.fbuf);
    vec(it.halo);
    vec(it.br.runs);
    vec(it.br.cell_loc);
    vec(it.br.face_loc);
    vec(it.br.face_code);
  }
  brick_body<T, D, N1, CELLS>(g - it.blk0[CELLS ? 3 : 1], it.br, (const T *)it.fbuf, (const T *)it.u, (T *)it.v, (T *)it.halo,
                       it.nh, tab, T(D == 3 ? it.sc.h : 1.0), SBM_PART_ALL);
}

template <typename T, int D>
__global__ __launch_bounds__(256) void halo_reduce_batch_kernel(const BatchItem *__restrict__ items,
                                                                const int32_t *__restrict__ blk_item) {
  const int g = blockIdx.x;
  const BatchItem it = batch_item(items, blk_item[g]);
  halo_reduce_body<T, D, false>(g - it.blk0[2], it.nh, it.halo_dof, it.halo_mask, (const T *)it.halo, (T *)it.v);
}

template <typename T, int D, int N1, int EPB>
__global__ __launch_bounds__(256, 4) void sbm_face_cg_batch_kernel(const BatchItem *__restrict__ items,
                                                                   const int32_t *__restrict__ blk_item,
                                                                   KTab<T, N1> tab) {
  const int g = xcd_block();
  const BatchItem it = batch_item(items, blk_item[g]);
  sbm_face_cg_body<T, D, N1, EPB>(g - it.blk0[0], it.nf, it.face_code, it.face_runs, it.face_xi,
                                  (const T *)it.u, (T *)it.fbuf, tab, it.sc);
}

template <typename T, int D, int N1>
__global__ __launch_bounds__(256) void sbm_face_dg_batch_kernel(const BatchItem *__restrict__ items,
                                                                const int32_t *__restrict__ blk_item,
                                                                KTab<T, N1> tab) {
  using S = BatchShape<T, D, N1>;
  const int g = xcd_block();
  const BatchItem it = batch_item(items, blk_item[g]);
  const int b = g - it.blk0[0];
  if constexpr (S::SLAB)
    sbm_face_slab_body<T, N1, S::EFD>(b, it.nf, it.face_cell, it.face_code, it.face_xi, (const T *)it.u, (T *)it.fbuf,
                                      tab, it.sc);
  else
    sbm_face_body<T, D, N1, S::EFD>(b, it.nf, it.face_cell, it.face_code, it.face_xi, (const T *)it.u,
                                    (T *)it.fbuf, tab, it.sc);
}

template <typename T, int D, int N1, int EPB>
__global__ __launch_bounds__(256) void dg_cell_batch_kernel(const BatchItem *__restrict__ items,
                                                            const int32_t *__restrict__ blk_item, KTab<T, N1> tab) {
  const int g = xcd_block();
  const BatchItem it = batch_item(items, blk_item[g]);
  const int b = g - it.blk0[1];
  const T scale = T(D == 3 ? it.sc.h : 1.0);
  dg_cell_body<T, D, N1, EPB>(b, it.nc, it.nbr, (const T *)it.u, (const T *)it.fbuf, (T *)it.v, tab, it.sc,
                                scale, SBM_PART_ALL);
}

// Workgroups of each stage for one item (faces: 0 when the item's surrogate faces are computed
// elsewhere, i.e. by a truncated extension).
template <typename T, int D, int N1>
void batch_blocks_impl(const sbm_ctx *c, bool own_faces, bool few, int32_t nb[4]) {
  using S = BatchShape<T, D, N1>;
  const int ec = few ? S::EC1 : S::EC;
  const int64_t nf = own_faces ? c->n_sbm : 0;
  if (c->disc == SBM_CG) {
    nb[0] = (int32_t)((nf + S::EF - 1) / S::EF);
    nb[1] = c->by_cells ? 0 : (int32_t)c->n_bricks;
    nb[3] = c->by_cells ? (int32_t)c->n_bricks : 0;
    nb[2] = (int32_t)((c->n_halo_dofs + kHaloPerThread * 256 - 1) / (kHaloPerThread * 256));
  } else {
    nb[0] = (int32_t)((nf + S::EFD - 1) / S::EFD);
    nb[1] = (int32_t)((c->n_cells + ec - 1) / ec);
    nb[2] = nb[3] = 0;
  }
}

template <typename T, int D, int N1>
hipError_t batch_launch_impl(const BatchGroup &g_, const unsigned char *base, hipStream_t s, int stages) {
  BatchGroup g = g_;
  for (int k = 0; k < 4; ++k)
    if (!((stages >> k) & 1)) g.nblk[k] = 0;
  using S = BatchShape<T, D, N1>;
  const KTab<T, N1> tab = make_ktab<T, N1>(g.first->rules);
  const BatchItem *items = reinterpret_cast<const BatchItem *>(base + g.off_items);
  const int32_t *bi[4];
  for (int k = 0; k < 4; ++k) bi[k] = reinterpret_cast<const int32_t *>(base + g.off_blk[k]);
  if (g.first->disc == SBM_CG) {
    if (g.nblk[0] > 0)
      hipLaunchKernelGGL((sbm_face_cg_batch_kernel<T, D, N1, S::EF>), dim3(g.nblk[0]), dim3(S::EF * S::NP), 0, s,
                         items, bi[0], tab);
    // the bricks of either form: two launches between one of the faces and one of the boundary sums (a
    // chain of its own for each form took 110 against 99 us for 6 balls of 16^3 to 52^3 Q4, FP64)
    auto bricks = [&](auto by_cells, int k) {
      constexpr bool CELLS = decltype(by_cells)::value;
      if (g.nblk[k] > 0)
        hipLaunchKernelGGL((brick_batch_kernel<T, D, N1, CELLS>), dim3(g.nblk[k]), dim3(BrickCfg<T, D, N1, CELLS>::NT),
                           0, s, items, bi[k], tab);
    };
    if constexpr (has_sweeps<D, N1>()) bricks(std::false_type{}, 1);
    constexpr int SPLIT = tile_split<D, N1>();
    if constexpr (SPLIT > 1) {
      if (g.nblk[3] > tile_split_from<T, N1>()) {
        hipLaunchKernelGGL((brick_split_batch_kernel<T, D, N1>), dim3(g.nblk[3]), dim3(TileBrickCfg<T, D, N1, SPLIT>::NT),
                           0, s, items, bi[3], tab);
        g.nblk[3] = 0;
      }
    }
    bricks(std::true_type{}, 3);
    if (g.nblk[2] > 0)
      hipLaunchKernelGGL((halo_reduce_batch_kernel<T, D>), dim3(g.nblk[2]), dim3(256), 0, s, items, bi[2]);
  } else {
    if (g.nblk[0] > 0)
      hipLaunchKernelGGL((sbm_face_dg_batch_kernel<T, D, N1>), dim3(g.nblk[0]), dim3(S::TFD), 0, s, items, bi[0], tab);
    auto cells = [&](auto epb) {
      constexpr int E = decltype(epb)::value;
      if (g.nblk[1] > 0)
        hipLaunchKernelGGL((dg_cell_batch_kernel<T, D, N1, E>), dim3(g.nblk[1]), dim3(E * S::NP), 0, s, items, bi[1], tab);
    };
    if (g.few)
      cells(std::integral_constant<int, S::EC1>{});
    else
      cells(std::integral_constant<int, S::EC>{});
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// Diagonal of A (for Jacobi preconditioning), one thread per (entity, local DoF):
//   cell:  h^(d-2) sum_k K_ii(axis k) prod_{m != k} M_ii(axis m)            (same every cell)
//   DG interior face (a, s) of K:  sum_q w_q (sigma_F psi_i^2 - psi_i dpsi_i/dn_K)
//   surrogate face:  sum_q w_q [ -dn psi_i psi_i(x~) - dn psi_i psi_i(x) + sigma psi_i(x) psi_i(x~) ]
// with psi_i(x~) on the face Gauss points and psi_i(x) at the shifted points.  Computed
// once per solve, so it uses plain loops and global atomics.
// ------------------------------------------------------------------------------------
template <typename T, int D, int N1>
__global__ void diag_cell_kernel(int n_cells, int disc_dg, const int32_t *__restrict__ runs,
                                 const int32_t *__restrict__ nbr, T *__restrict__ diag, KTab<T, N1> tab, KScal sc,
                                 T scale) {
  constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB, P = N1 - 1;
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid >= (int64_t)n_cells * NB) return;
  const int cell = (int)(gid / NB), i = (int)(gid % NB);
  const int ik[3] = {i % N1, (i / N1) % N1, (D == 3) ? i / (N1 * N1) : 0};
  double val = 0.0;
  for (int k = 0; k < D; ++k) {
    double t = tab.K[ik[k] * N1 + ik[k]];
    for (int m = 0; m < D; ++m)
      if (m != k) t *= tab.M[ik[m] * N1 + ik[m]];
    val += t;
  }
  val *= (double)scale;
  if (disc_dg) {
    const double h = sc.h;
    for (int code = 0; code < 2 * D; ++code) {
      if (nbr[(int64_t)cell * 2 * D + code] < 0) continue;
      const int a = code >> 1, s = code & 1;
      if (ik[a] != s * P) {
        // psi_i vanishes on this face: only the derivative term times psi_i = 0
        continue;
      }
      const double sgn = s ? 1.0 : -1.0;
      const double ds = s ? (double)tab.D1[ik[a]] : (double)tab.D0[ik[a]];
      for (int q = 0; q < NP; ++q) {
        const int qt[2] = {q % N1, (D == 3) ? q / N1 : 0};
        double tang = 1.0, om = 1.0;
        int t = 0;
        for (int m = 0; m < D; ++m) {
          if (m == a) continue;
          tang *= (double)tab.N[qt[t] * N1 + ik[m]];
          om *= (double)tab.w[qt[t]] * h;
          ++t;
        }
        val += om * (sc.sigma_f * tang * tang - tang * sgn / h * ds * tang);
      }
    }
    diag[(int64_t)cell * NB + i] = (T)val;
  } else {
    atomic_add(diag + runs[(int64_t)cell * NP + i / N1] + i % N1, (T)val);
  }
}

template <typename T, int D, int N1>
__global__ void diag_face_kernel(int n_faces, int disc_dg, const int32_t *__restrict__ face_cell,
                                 const int32_t *__restrict__ face_code, const double *__restrict__ face_xi,
                                 const int32_t *__restrict__ runs, T *__restrict__ diag, KTab<T, N1> tab, KScal sc) {
  constexpr int NP = Shape<D, N1>::NP, NB = Shape<D, N1>::NB, P = N1 - 1;
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid >= (int64_t)n_faces * NB) return;
  const int f = (int)(gid / NB), i = (int)(gid % NB);
  const int cell = face_cell[f], code = face_code[f], a = code >> 1, s = code & 1;
  const int ik[3] = {i % N1, (i / N1) % N1, (D == 3) ? i / (N1 * N1) : 0};
  const double h = sc.h, sgn = s ? 1.0 : -1.0;
  const double ds = s ? (double)tab.D1[ik[a]] : (double)tab.D0[ik[a]];
  double val = 0.0;
  for (int q = 0; q < NP; ++q) {
    const int qt[2] = {q % N1, (D == 3) ? q / N1 : 0};
    double tang = 1.0, om = 1.0;
    int t = 0;
    for (int m = 0; m < D; ++m) {
      if (m == a) continue;
      tang *= (double)tab.N[qt[t] * N1 + ik[m]];
      om *= (double)tab.w[qt[t]] * h;
      ++t;
    }
    const double vt = (ik[a] == s * P) ? tang : 0.0;  // psi_i(x~_q)
    const double dn = sgn / h * ds * tang;            // d psi_i / dn~ (x~_q)
    double vs = 1.0;                                  // psi_i(x_q), shifted point
    const double *xq = face_xi + ((int64_t)f * NP + q) * D;
    for (int m = 0; m < D; ++m) {
      double l[N1];
      lagrange_at<N1>(tab.z, tab.cinv, xq[m], l);
      vs *= l[ik[m]];
    }
    val += om * (-dn * vt - dn * vs + sc.sigma_gamma * vs * vt);
  }
  const int64_t dof = disc_dg ? (int64_t)cell * NB + i : (int64_t)runs[(int64_t)cell * NP + i / N1] + i % N1;
  atomic_add(diag + dof, (T)val);
}

template <typename T, int D, int N1>
hipError_t diag_impl(const sbm_ctx *c, T *diag, hipStream_t s) {
  constexpr int NB = Shape<D, N1>::NB;
  const KTab<T, N1> tab = make_ktab<T, N1>(c->rules);
  const KScal sc{c->h, c->sigma_gamma, c->sigma_f};
  const T scale = T(D == 3 ? c->h : 1.0);
  const int dg = c->disc == SBM_DG;
  hipError_t e = vec_fill(diag, c->n_dofs, 0.0, sizeof(T) == 8 ? SBM_F64 : SBM_F32, s);
  if (e != hipSuccess) return e;
  const int64_t nc = c->n_cells * NB, nf = c->n_sbm * NB;
  if (nc > 0)
    hipLaunchKernelGGL((diag_cell_kernel<T, D, N1>), dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s,
                       (int)c->n_cells, dg, c->d_runs, c->d_nbr, diag, tab, sc, scale);
  if (nf > 0)
    hipLaunchKernelGGL((diag_face_kernel<T, D, N1>), dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s,
                       (int)c->n_sbm, dg, c->d_face_cell, c->d_face_code, c->d_face_xi, c->d_runs, diag, tab, sc);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t diag_dim(const sbm_ctx *c, T *diag, hipStream_t s) {
  switch (c->p) {
    case 1: return diag_impl<T, D, 2>(c, diag, s);
    case 2: return diag_impl<T, D, 3>(c, diag, s);
    case 3: return diag_impl<T, D, 4>(c, diag, s);
    case 4: return diag_impl<T, D, 5>(c, diag, s);
    case 5: return diag_impl<T, D, 6>(c, diag, s);
    case 6: return diag_impl<T, D, 7>(c, diag, s);
    case 7: return diag_impl<T, D, 8>(c, diag, s);
    case 8: return diag_impl<T, D, 9>(c, diag, s);
  }
  return hipErrorInvalidValue;
}

#define SBM_P_SWITCH(P_, CALL)     \
  switch (P_) {                    \
    case 1: return CALL(2);        \
    case 2: return CALL(3);        \
    case 3: return CALL(4);        \
    case 4: return CALL(5);        \
    case 5: return CALL(6);        \
    case 6: return CALL(7);        \
    case 7: return CALL(8);        \
    case 8: return CALL(9);        \
  }

template <typename T, int D>
bool batch_blocks_dim(const sbm_ctx *c, bool own_faces, bool few, int32_t nb[4]) {
#define SBM_BB(N1_) (batch_blocks_impl<T, D, N1_>(c, own_faces, few, nb), true)
  SBM_P_SWITCH(c->p, SBM_BB)
#undef SBM_BB
  return false;
}

template <typename T, int D>
hipError_t batch_launch_dim(const BatchGroup &g, const unsigned char *base, hipStream_t s, int stages) {
#define SBM_BL(N1_) batch_launch_impl<T, D, N1_>(g, base, s, stages)
  SBM_P_SWITCH(g.first->p, SBM_BL)
#undef SBM_BL
  return hipErrorInvalidValue;
}
#undef SBM_P_SWITCH

template <typename T, int D>
hipError_t apply_dim(const sbm_ctx *c, const T *u, T *v, int parts, hipStream_t s, const Scratch &scr) {
  switch (c->p) {
    case 1: return apply_impl<T, D, 2>(c, u, v, parts, s, scr);
    case 2: return apply_impl<T, D, 3>(c, u, v, parts, s, scr);
    case 3: return apply_impl<T, D, 4>(c, u, v, parts, s, scr);
    case 4: return apply_impl<T, D, 5>(c, u, v, parts, s, scr);
    case 5: return apply_impl<T, D, 6>(c, u, v, parts, s, scr);
    case 6: return apply_impl<T, D, 7>(c, u, v, parts, s, scr);
    case 7: return apply_impl<T, D, 8>(c, u, v, parts, s, scr);
    case 8: return apply_impl<T, D, 9>(c, u, v, parts, s, scr);
  }
  return hipErrorInvalidValue;
}

}  // namespace

bool brick_by_cells(int dim, int p, int64_t n_cells) { return n_cells <= kCellsMax[dim - 2][p]; }

void brick_dims(int dim, int p, bool by_cells, int *bx, int *by, int *bz) {
#define SBM_BD(D_, P_, C_)                     \
  if (dim == D_ && p == P_ && by_cells == C_) { \
    *bx = BrickDims<D_, P_, C_>::BX;           \
    *by = BrickDims<D_, P_, C_>::BY;           \
    *bz = BrickDims<D_, P_, C_>::BZ;           \
    return;                                    \
  }
#define SBM_BD2(D_, P_) SBM_BD(D_, P_, true) SBM_BD(D_, P_, false)
  SBM_BD2(2, 1) SBM_BD2(2, 2) SBM_BD2(2, 3) SBM_BD2(2, 4) SBM_BD2(2, 5) SBM_BD2(2, 6) SBM_BD2(2, 7) SBM_BD2(2, 8)
  SBM_BD2(3, 1) SBM_BD2(3, 2) SBM_BD2(3, 3) SBM_BD2(3, 4) SBM_BD2(3, 5) SBM_BD2(3, 6) SBM_BD2(3, 7) SBM_BD2(3, 8)
#undef SBM_BD2
#undef SBM_BD
  *bx = *by = *bz = 1;
}

hipError_t launch_diagonal(const sbm_ctx *c, void *diag, int prec, hipStream_t s) {
  if (prec == SBM_F64)
    return c->dim == 3 ? diag_dim<double, 3>(c, (double *)diag, s) : diag_dim<double, 2>(c, (double *)diag, s);
  return c->dim == 3 ? diag_dim<float, 3>(c, (float *)diag, s) : diag_dim<float, 2>(c, (float *)diag, s);
}

size_t apply_scratch_bytes(const sbm_ctx *c, int prec) {
  const size_t s = prec == SBM_F64 ? sizeof(double) : sizeof(float);
  auto up = [](size_t b) { return (b + 255) / 256 * 256; };
  const size_t halo = c->disc == SBM_CG ? ((size_t)1 << c->dim) * (size_t)c->n_halo_dofs * s : 0;
  const size_t fbuf = (size_t)c->n_sbm * 2 * (size_t)c->nq_face * s;
  return up(halo) + up(fbuf);
}

hipError_t batch_group_build(BatchGroup &g, const std::vector<const sbm_ctx *> &cs,
                             const std::vector<const void *> &u, const std::vector<void *> &v,
                             const std::vector<int> &own_faces, std::vector<unsigned char> &image) {
  const sbm_ctx *c0 = cs.empty() ? nullptr : cs[0];
  if (!c0 || u.size() != cs.size() || v.size() != cs.size() || own_faces.size() != cs.size())
    return hipErrorInvalidValue;
  g.first = c0;
  g.n_items = (int)cs.size();
  std::vector<BatchItem> items(cs.size());
  std::vector<int32_t> blk[4];
  int64_t tot[4] = {0, 0, 0, 0};
  auto blocks = [&](const sbm_ctx *c, bool own, bool few, int32_t (&nb)[4]) {
    return g.prec == SBM_F64 ? (c->dim == 3 ? batch_blocks_dim<double, 3>(c, own, few, nb)
                                            : batch_blocks_dim<double, 2>(c, own, few, nb))
                             : (c->dim == 3 ? batch_blocks_dim<float, 3>(c, own, few, nb)
                                            : batch_blocks_dim<float, 2>(c, own, few, nb));
  };
  int64_t full = 0;
  for (size_t i = 0; i < cs.size(); ++i) {
    const sbm_ctx *c = cs[i];
    if (c->disc != c0->disc || c->dim != c0->dim || c->p != c0->p) return hipErrorInvalidValue;
    int32_t nb[4] = {0, 0, 0, 0};
    if (!blocks(c, false, false, nb)) return hipErrorInvalidValue;
    full += nb[1];
  }
  g.few = c0->disc == SBM_DG && full < two_per_cu();
  for (size_t i = 0; i < cs.size(); ++i) {
    const sbm_ctx *c = cs[i];
    int32_t nb[4] = {0, 0, 0, 0};
    if (!blocks(c, own_faces[i] != 0, g.few, nb)) return hipErrorInvalidValue;
    BatchItem &it = items[i];
    it.br = BrickArgs{c->d_brick_cell_off, c->d_brick_runs, c->d_brick_cell_loc, c->d_brick_face_off,
                      c->d_brick_face_loc, c->d_face_code,  c->d_brick_cell_face, c->d_row_base,       c->d_row_gmask,
                      c->d_row_bmask,      c->d_row_hbase,     c->d_row_hend};
    it.face_code = c->d_face_code;
    it.face_runs = c->d_face_runs;
    it.face_cell = c->d_face_cell;
    it.nbr = c->d_nbr;
    it.halo_dof = c->d_halo_dof;
    it.halo_mask = c->d_halo_mask;
    it.face_xi = c->d_face_xi;
    it.u = u[i];
    it.v = v[i];
    it.fbuf = c->d_fbuf;
    it.halo = c->d_halo;
    it.sc = KScal{c->h, c->sigma_gamma, c->sigma_f};
    it.nf = (int)c->n_sbm;
    it.nc = (int)c->n_cells;
    it.nh = (int)c->n_halo_dofs;
    for (int k = 0; k < 4; ++k) {
      it.blk0[k] = (int)tot[k];
      blk[k].insert(blk[k].end(), (size_t)nb[k], (int32_t)i);
      tot[k] += nb[k];
      if (tot[k] > INT32_MAX / 2) return hipErrorInvalidValue;
    }
  }
  auto put = [&image](const void *src, size_t bytes) {
    const size_t off = (image.size() + 255) / 256 * 256;
    image.resize(off + std::max<size_t>(bytes, 4));
    if (bytes) std::memcpy(image.data() + off, src, bytes);
    return off;
  };
  g.off_items = put(items.data(), items.size() * sizeof(BatchItem));
  for (int k = 0; k < 4; ++k) {
    g.nblk[k] = (int)tot[k];
    g.off_blk[k] = put(blk[k].data(), blk[k].size() * sizeof(int32_t));
  }
  return hipSuccess;
}

hipError_t launch_batch_group(const BatchGroup &g, const void *base, hipStream_t s, int stages) {
  const unsigned char *b = static_cast<const unsigned char *>(base);
  if (g.prec == SBM_F64)
    return g.first->dim == 3 ? batch_launch_dim<double, 3>(g, b, s, stages) : batch_launch_dim<double, 2>(g, b, s, stages);
  return g.first->dim == 3 ? batch_launch_dim<float, 3>(g, b, s, stages) : batch_launch_dim<float, 2>(g, b, s, stages);
}

hipError_t launch_apply(const sbm_ctx *c, const void *u, void *v, int prec, int parts, hipStream_t s,
                        const Scratch *scr) {
  Scratch use;
  use.halo = (scr && scr->halo) ? scr->halo : c->d_halo;
  use.fbuf = (scr && scr->fbuf) ? scr->fbuf : c->d_fbuf;
  if (prec == SBM_F64) {
    return c->dim == 3 ? apply_dim<double, 3>(c, (const double *)u, (double *)v, parts, s, use)
                       : apply_dim<double, 2>(c, (const double *)u, (double *)v, parts, s, use);
  }
  return c->dim == 3 ? apply_dim<float, 3>(c, (const float *)u, (float *)v, parts, s, use)
                     : apply_dim<float, 2>(c, (const float *)u, (float *)v, parts, s, use);
}

}  // namespace sbm
