// Truncated-Taylor extension of the shifted boundary operator.
//
// Sec. 2.1 transfers the boundary value from the true boundary to the surrogate one by a Taylor
// expansion of the solution about the surrogate point x~ along the shift d = x - x~.  The
// default operator evaluates the face's cell polynomial at the shifted point, which is that
// expansion to all orders (it terminates for a polynomial).  This file provides the expansion
// kept to total order m:
//     E_m u(x~) = sum over |alpha| <= m of D^alpha u_K(x~) d^alpha / alpha!,
// in reference coordinates of the face's own cell (D_x^alpha d^alpha = D_xi^alpha delta^alpha,
// delta = xi - xi~).  m = 1 is the value-plus-gradient form; m >= d p is the full extension.
//
// Only the surrogate-face term changes: with an order set on a handle, sbm_face_taylor_kernel
// leaves each face's (Rv, Rg) per face node in the handle's face buffer, and the default cell
// kernels (brick kernel for CG, cell kernel for DG) then expand and merge them in face order,
// exactly as for the full extension.  The diagonal is the default one plus a correction of its
// surrogate-face term.
#include "sbm_internal.h"

namespace sbm {
namespace {

constexpr int kTaylorThreads = 256;

// FP64 1D data on [0,1] for the face kernels (kernel argument, by value).
struct TaylorTab {
  double z[kMaxN1], cinv[kMaxN1];  // GLL nodes, 1 / prod_{l != j} (z_j - z_l)
  double g[kMaxN1], w[kMaxN1];     // Gauss points and weights of the face rule
  double N[kMaxN1 * kMaxN1];       // N[q N1 + j] = l_j(g_q)
  double D0[kMaxN1], D1[kMaxN1];   // l'_j(0), l'_j(1)
};

TaylorTab make_taylor_tab(const Rules1D &r) {
  TaylorTab t{};
  const int n1 = r.p + 1;
  for (int j = 0; j < n1; ++j) {
    t.z[j] = r.z[j];
    t.cinv[j] = r.cinv[j];
    t.g[j] = r.g[j];
    t.w[j] = r.w[j];
    t.D0[j] = r.D0[j];
    t.D1[j] = r.D1[j];
  }
  for (int i = 0; i < n1 * n1; ++i) t.N[i] = r.N[i];
  return t;
}

// Taylor terms of the 1D basis function j about x0: c[k] = l_j^(k)(x0) dlt^k / k!, k <= p.
// They are the coefficients of t^k in
// l_j(x0 + t dlt) = cinv_j prod_{l != j} (x0 - z_l + t dlt): the p linear factors (x0 - z_l) + s
// are multiplied out in s = t dlt (one multiply-add per coefficient and factor), and coefficient k
// is then scaled by cinv_j dlt^k.
template <int N1>
__device__ __forceinline__ void taylor_terms(const TaylorTab &tt, int j, double x0, double dlt, double (&c)[N1]) {
  double poly[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) poly[k] = k == 0 ? 1.0 : 0.0;
#pragma unroll
  for (int l = 0; l < N1; ++l) {
    if (l == j) continue;
    const double a = x0 - tt.z[l];
#pragma unroll
    for (int k = N1 - 1; k >= 1; --k) poly[k] = a * poly[k] + poly[k - 1];
    poly[0] *= a;
  }
  double scale = tt.cinv[j];
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    c[k] = scale * poly[k];
    scale *= dlt;
  }
}

// Reference coordinates of the surrogate point of face point q on face (a, s): xi~_a = s, the
// tangential axes (lower one fastest) at the Gauss points.
template <int D, int N1>
__device__ __forceinline__ void surrogate_point(const TaylorTab &tt, int a, int s, int q, double (&x0)[D]) {
  int qq = q;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    if (k == a) {
      x0[k] = (double)s;
    } else {
      x0[k] = tt.g[qq % N1];
      qq /= N1;
    }
  }
}

// Local DoF i of the face's cell -> global DoF (CG through the cell's x-run bases).
template <int D, int N1>
__device__ __forceinline__ int64_t local_dof(int disc_dg, const int32_t *__restrict__ runs, int cell, int i) {
  constexpr int NP = D == 3 ? N1 * N1 : N1, NB = NP * N1;
  return disc_dg ? (int64_t)cell * NB + i : (int64_t)runs[(int64_t)cell * NP + i / N1] + i % N1;
}

// Slabs of the cell that split a face point's evaluation of E_m u over threads: p+1 where
// (p+1)^d threads fit in a workgroup, else 1 (one thread takes every slab).
template <int D, int N1>
constexpr int taylor_slabs() {
  return (D == 3 ? N1 * N1 * N1 : N1 * N1) <= kTaylorThreads ? N1 : 1;
}

// One workgroup per surrogate face (Eq. (1) face terms with E replaced by E_m):
//   row_i = sum_q w_q [ -(dn u)(x~_q) psi_i(x~_q) - (dn psi_i)(x~_q) E_m u(x~_q)
//                       + sigma_Gam E_m u(x~_q) psi_i(x~_q) ],
// added into v.  Phase 1, thread (q, slab): the Taylor terms of face point q along the d axes,
// then its slab's share of E_m u (the cell values contracted axis by axis with the order sum
// kept <= m) and of the normal derivative at x~_q; the slab shares are added in slab order.
// Phase 2, one thread per face node: Rv = sum_q psi(x~_q) w_q (sigma E_m u - dn u) and
// Rg = -sum_q psi(x~_q) w_q E_m u (2s-1)/h over the tangential basis, stored per face node in
// fbuf (fbuf[f][0][t], fbuf[f][1][t]); the cell kernels add the face's rows (Rv on the face's
// own nodes plus Rg times the normal derivative of the row's 1D function) in a fixed order, as
// for the full extension.  FP64 inside; the 1D tables are staged in LDS.  All p+1
// Taylor orders per axis; launches with m <= 2 take sbm_face_taylor_low_kernel.
template <typename T, int D, int N1>
__global__ __launch_bounds__(kTaylorThreads) void sbm_face_taylor_kernel(
    int n_faces, int disc_dg, int m, const int32_t *__restrict__ face_cell, const int32_t *__restrict__ face_code,
    const double *__restrict__ face_xi, const int32_t *__restrict__ runs, const T *__restrict__ u,
    T *__restrict__ fbuf, TaylorTab tt, double h, double sigma) {
  constexpr int NP = D == 3 ? N1 * N1 : N1, NB = NP * N1, S = taylor_slabs<D, N1>();
  __shared__ double su[NB];
  __shared__ double sN[N1 * N1], sDs[N1], sw[N1];
  __shared__ double pe[S][NP], pd[S][NP];  // slab shares of E_m u and of the normal derivative
  __shared__ double sA[NP], sB[NP];
  const int f = blockIdx.x;
  if (f >= n_faces) return;
  const int cell = face_cell[f], code = face_code[f], a = code >> 1, s = code & 1;
  const double sgn = s ? 1.0 : -1.0;
  for (int i = threadIdx.x; i < NB; i += blockDim.x) su[i] = (double)u[local_dof<D, N1>(disc_dg, runs, cell, i)];
  for (int i = threadIdx.x; i < N1 * N1; i += blockDim.x) sN[i] = tt.N[i];
  if (threadIdx.x < N1) {
    sDs[threadIdx.x] = s ? tt.D1[threadIdx.x] : tt.D0[threadIdx.x];
    sw[threadIdx.x] = tt.w[threadIdx.x];
  }
  __syncthreads();
  // tangential axes of the face, lower one first (face point q = qb + N1 qc)
  const int tb = a == 0 ? 1 : 0;  // (the upper tangential axis is the remaining one)
  for (int t = threadIdx.x; t < NP * S; t += blockDim.x) {
    const int q = t % NP, slab = t / NP;
    const int qb = q % N1, qc = D == 3 ? q / N1 : 0;
    double x0[D], dl[D];
    surrogate_point<D, N1>(tt, a, s, q, x0);
#pragma unroll
    for (int k = 0; k < D; ++k) dl[k] = face_xi[((int64_t)f * NP + q) * D + k] - x0[k];
    // c[k][i][j]: order-j Taylor term of basis function i along axis k < d-1 (the last axis
    // is the slab axis: only the slab's own function is needed, cl below)
    double c[D - 1][N1][N1];
#pragma unroll
    for (int k = 0; k < D - 1; ++k)
#pragma unroll
      for (int i = 0; i < N1; ++i) taylor_terms<N1>(tt, i, x0[k], dl[k], c[k][i]);
    // factor of local index i along axis k in the normal derivative at x~_q
    auto dfac = [&](int k, int i) {
      return k == a ? sDs[i] : sN[(k == tb ? qb : qc) * N1 + i];
    };
    double eu = 0.0, dn = 0.0;
    for (int il = slab; il < N1; il += S) {  // slab il: last local index (i2 in 3D, i1 in 2D)
      double cl[N1];
      taylor_terms<N1>(tt, il, x0[D - 1], dl[D - 1], cl);
      if constexpr (D == 3) {
        double b[N1][N1];  // b[j0][j1] = sum_{i0,i1} c0[i0][j0] c1[i1][j1] u[i0,i1,il]
#pragma unroll
        for (int j0 = 0; j0 < N1; ++j0)
#pragma unroll
          for (int j1 = 0; j1 < N1; ++j1) b[j0][j1] = 0.0;
        const double f2 = dfac(2, il);
#pragma unroll
        for (int i1 = 0; i1 < N1; ++i1) {
          double r[N1];
          double g = 0.0;
          const double f1 = dfac(1, i1);
#pragma unroll
          for (int j0 = 0; j0 < N1; ++j0) r[j0] = 0.0;
#pragma unroll
          for (int i0 = 0; i0 < N1; ++i0) {
            const double uv = su[i0 + N1 * i1 + NP * il];
            g += dfac(0, i0) * uv;
#pragma unroll
            for (int j0 = 0; j0 < N1; ++j0) r[j0] += c[0][i0][j0] * uv;
          }
          dn += f2 * f1 * g;
#pragma unroll
          for (int j0 = 0; j0 < N1; ++j0)
#pragma unroll
            for (int j1 = 0; j1 < N1; ++j1) b[j0][j1] += c[1][i1][j1] * r[j0];
        }
        // sum over j0 + j1 + j2 <= m of cl[j2] b[j0][j1]: b summed along its anti-diagonals
        // (j0 + j1 = k) first, then each order j2 takes the diagonals k <= m - j2
        double bd[2 * N1 - 1];
#pragma unroll
        for (int k = 0; k < 2 * N1 - 1; ++k) bd[k] = 0.0;
#pragma unroll
        for (int j0 = 0; j0 < N1; ++j0)
#pragma unroll
          for (int j1 = 0; j1 < N1; ++j1) bd[j0 + j1] += b[j0][j1];
#pragma unroll
        for (int j2 = 0; j2 < N1; ++j2) {
          double t = 0.0;
#pragma unroll
          for (int k = 0; k < 2 * N1 - 1; ++k)
            if (k + j2 <= m) t += bd[k];
          eu += cl[j2] * t;
        }
      } else {
        double g = 0.0;
        const double f1 = dfac(1, il);
#pragma unroll
        for (int j0 = 0; j0 < N1; ++j0) {
          double acc = 0.0;
#pragma unroll
          for (int i0 = 0; i0 < N1; ++i0) acc += c[0][i0][j0] * su[i0 + N1 * il];
#pragma unroll
          for (int j1 = 0; j1 < N1; ++j1)
            if (j0 + j1 <= m) eu += cl[j1] * acc;
        }
#pragma unroll
        for (int i0 = 0; i0 < N1; ++i0) g += dfac(0, i0) * su[i0 + N1 * il];
        dn += f1 * g;
      }
    }
    pe[slab][q] = eu;
    pd[slab][q] = dn;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < NP; q += blockDim.x) {
    double eu = 0.0, dn = 0.0;
#pragma unroll
    for (int k = 0; k < S; ++k) {
      eu += pe[k][q];
      dn += pd[k][q];
    }
    dn *= sgn / h;
    double om = sw[q % N1] * h;
    if constexpr (D == 3) om *= sw[q / N1] * h;
    sA[q] = om * (sigma * eu - dn);  // tested against psi(x~_q)
    sB[q] = -om * eu * sgn / h;      // tested against the normal derivative's 1D factor
  }
  __syncthreads();
  for (int t = threadIdx.x; t < NP; t += blockDim.x) {
    const int jb = t % N1, jc = D == 3 ? t / N1 : 0;
    double rv = 0.0, rg = 0.0;
    for (int q = 0; q < NP; ++q) {
      const double tang = sN[(q % N1) * N1 + jb] * (D == 3 ? sN[(q / N1) * N1 + jc] : 1.0);
      rv += tang * sA[q];
      rg += tang * sB[q];
    }
    fbuf[(int64_t)f * 2 * NP + t] = (T)rv;
    fbuf[(int64_t)f * 2 * NP + NP + t] = (T)rg;
  }
}

// Low orders (m <= M, M = 1 or 2) by sum factorisation.  The derivatives are taken at the surrogate
// points, which form a tensor grid on the face, so D^alpha u_K there is: the normal derivatives of
// order a at the face nodes (T_a, from the nodes' lines along the normal), then the 1D basis
// derivatives of order b at the lower tangential Gauss points (Y_ab), then those of order c at the
// upper ones; each face point sums delta^alpha / alpha! times them over a + b + c <= m.  The normal
// derivative of Eq. (1) is the a = 1 term without the tangential ones.  About 60 multiply-adds per
// face point at M = 1 (180 at M = 2) against 600 (2,800) when every point contracts the whole cell,
// and no cell values in LDS.  One thread per face node and face point, EPB faces per workgroup; FP64
// inside.  Bound by latency (five short phases); 64^3 Q4 sphere, 10,176 faces, m = 1, FP64: 32.4 -> 11.8 us.
// (sized by degree and order: at 2.5 KB for all of them, the launch of 2D Q2 cost the host 1 us more)
template <int N1, int M>
struct TaylorLowTab {
  double G[M + 1][N1 * N1];  // G[k][q N1 + j] = l_j^(k)(g_q) / k!
  double E[2][M + 1][N1];    // E[s][k][j] = l_j^(k)(s) / k!
  double g[N1], w[N1];       // Gauss points and weights
};

// l_j^(k)(x) / k!, k <= 2: coefficients of prod_{l != j} (x - z_l + t) / (z_j - z_l)
void lagrange_jet(const Rules1D &r, int j, double x, double (&c)[3]) {
  c[0] = r.cinv[j];
  c[1] = c[2] = 0.0;
  for (int l = 0; l <= r.p; ++l) {
    if (l == j) continue;
    const double a = x - r.z[l];
    c[2] = a * c[2] + c[1];
    c[1] = a * c[1] + c[0];
    c[0] *= a;
  }
}

template <int N1, int M>
TaylorLowTab<N1, M> make_taylor_low_tab(const Rules1D &r) {
  TaylorLowTab<N1, M> t;
  double c[3];
  for (int j = 0; j < N1; ++j) {
    for (int q = 0; q < N1; ++q) {
      lagrange_jet(r, j, r.g[q], c);
      for (int k = 0; k <= M; ++k) t.G[k][q * N1 + j] = c[k];
    }
    for (int s = 0; s < 2; ++s) {
      lagrange_jet(r, j, (double)s, c);
      for (int k = 0; k <= M; ++k) t.E[s][k][j] = c[k];
    }
    t.g[j] = r.g[j];
    t.w[j] = r.w[j];
  }
  return t;
}

template <int D, int N1>
constexpr int low_faces_per_block() {
  return kTaylorThreads / (D == 3 ? N1 * N1 : N1);
}

// Index of the pair (a, b), a + b <= M, in the order (0,0) .. (0,M), (1,0) ..
template <int M>
__host__ __device__ constexpr int pair_ix(int a, int b) {
  return a * (M + 1) - a * (a - 1) / 2 + b;
}

template <typename T, int D, int N1, int M>
__global__ __launch_bounds__(kTaylorThreads) void sbm_face_taylor_low_kernel(
    int n_faces, int disc_dg, int m, const int32_t *__restrict__ face_cell, const int32_t *__restrict__ face_code,
    const double *__restrict__ face_xi, const int32_t *__restrict__ face_runs, const T *__restrict__ u,
    T *__restrict__ fbuf, TaylorLowTab<N1, M> tt, double h, double sigma) {
  constexpr int NP = D == 3 ? N1 * N1 : N1, NB = NP * N1, EPB = low_faces_per_block<D, N1>(), P = N1 - 1;
  constexpr int NY = pair_ix<M>(M, 0) + 1;  // pairs (a, b) with a + b <= M
  __shared__ double sG[M + 1][N1 * N1], sE[2][M + 1][N1], sg[N1], sw[N1];
  __shared__ double sT[EPB][M + 1][NP], sY[EPB][D == 3 ? NY : 1][NP];
  for (int i = threadIdx.x; i < (M + 1) * N1 * N1; i += blockDim.x) sG[i / (N1 * N1)][i % (N1 * N1)] = tt.G[i / (N1 * N1)][i % (N1 * N1)];
  for (int i = threadIdx.x; i < 2 * (M + 1) * N1; i += blockDim.x)
    sE[i / ((M + 1) * N1)][i / N1 % (M + 1)][i % N1] = tt.E[i / ((M + 1) * N1)][i / N1 % (M + 1)][i % N1];
  if (threadIdx.x < N1) {
    sg[threadIdx.x] = tt.g[threadIdx.x];
    sw[threadIdx.x] = tt.w[threadIdx.x];
  }
  const int le = threadIdx.x / NP, t = threadIdx.x - le * NP;
  const int f = blockIdx.x * EPB + le;
  const bool act = f < n_faces;
  const int code = act ? face_code[f] : 0, a = code >> 1, s = code & 1;
  const int tb = t % N1, tc = D == 3 ? t / N1 : 0;  // node (jb, jc), later point (qb, qc)
  // the node's line along the face normal: local DoF i = run * N1 + position in the run
  const int64_t cell0 = disc_dg && act ? (int64_t)face_cell[f] * NB : 0;
  const int32_t *const runs = face_runs + (act ? (int64_t)f * NP : 0);
  double x[N1];
#pragma unroll
  for (int i = 0; i < N1; ++i) {
    int run, at;
    if (D == 3) {
      run = a == 0 ? t : (a == 1 ? i + N1 * tc : tc + N1 * i);
      at = a == 0 ? i : tb;
    } else {
      run = a == 0 ? tb : i;
      at = a == 0 ? i : tb;
    }
    x[i] = act ? (double)u[disc_dg ? cell0 + run * N1 + at : (int64_t)runs[run] + at] : 0.0;
  }
  double dl[D];  // shift of the thread's face point: along the normal, lower, upper tangential axis
  {
    const double *xp = face_xi + (act ? ((int64_t)f * NP + t) * D : 0);
    double xi[D];
#pragma unroll
    for (int k = 0; k < D; ++k) xi[k] = act ? xp[k] : 0.0;
    dl[0] = xi[0];
    dl[1] = xi[1];
    if (a == 1) {
      dl[0] = xi[1];
      dl[1] = xi[0];
    }
    if constexpr (D == 3) {
      dl[2] = a == 2 ? xi[1] : xi[2];
      if (a == 2) {
        dl[0] = xi[2];
        dl[1] = xi[0];
      }
    }
  }
  __syncthreads();
  dl[0] -= (double)s;
  dl[1] -= sg[tb];
  if constexpr (D == 3) dl[2] -= sg[tc];
#pragma unroll
  for (int k = 0; k <= M; ++k) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < N1; ++i) v += sE[s][k][i] * x[i];
    sT[le][k][t] = k == 0 ? (s ? x[P] : x[0]) : v;
  }
  __syncthreads();
  // powers of the shift (order 0 only where m = 0)
  const double on1 = m >= 1 ? 1.0 : 0.0, on2 = m >= 2 ? 1.0 : 0.0;
  double eu = 0.0, dn = 0.0;
  if constexpr (D == 3) {
    // lower tangential axis: Y_ab at (qb, jc)
#pragma unroll
    for (int ka = 0; ka <= M; ++ka)
#pragma unroll
      for (int kb = 0; kb <= M - ka; ++kb) {
        double v = 0.0;
#pragma unroll
        for (int j = 0; j < N1; ++j) v += sG[kb][tb * N1 + j] * sT[le][ka][j + N1 * tc];
        sY[le][pair_ix<M>(ka, kb)][t] = v;
      }
    __syncthreads();
#pragma unroll
    for (int ka = 0; ka <= M; ++ka)
#pragma unroll
      for (int kb = 0; kb <= M - ka; ++kb)
#pragma unroll
        for (int kc = 0; kc <= M - ka - kb; ++kc) {
          double v = 0.0;
#pragma unroll
          for (int j = 0; j < N1; ++j) v += sG[kc][tc * N1 + j] * sY[le][pair_ix<M>(ka, kb)][tb + N1 * j];
          if (ka == 1 && kb == 0 && kc == 0) dn = v;
          const int k = ka + kb + kc;
          double w = k == 0 ? 1.0 : (k == 1 ? on1 : on2);
#pragma unroll
          for (int q = 0; q < ka; ++q) w *= dl[0];
#pragma unroll
          for (int q = 0; q < kb; ++q) w *= dl[1];
#pragma unroll
          for (int q = 0; q < kc; ++q) w *= dl[D - 1];
          eu += k == 0 ? v : w * v;
        }
  } else {
#pragma unroll
    for (int ka = 0; ka <= M; ++ka)
#pragma unroll
      for (int kb = 0; kb <= M - ka; ++kb) {
        double v = 0.0;
#pragma unroll
        for (int j = 0; j < N1; ++j) v += sG[kb][tb * N1 + j] * sT[le][ka][j];
        if (ka == 1 && kb == 0) dn = v;
        const int k = ka + kb;
        double w = k == 0 ? 1.0 : (k == 1 ? on1 : on2);
#pragma unroll
        for (int q = 0; q < ka; ++q) w *= dl[0];
#pragma unroll
        for (int q = 0; q < kb; ++q) w *= dl[1];
        eu += k == 0 ? v : w * v;
      }
  }
  const double sgn = s ? 1.0 : -1.0;
  dn *= sgn / h;
  double om = sw[tb] * h;
  if constexpr (D == 3) om *= sw[tc] * h;
  // integration to the face nodes of A (tested against psi) and B (against its normal derivative)
  double *const fa = sT[le][0], *const fb = sT[le][1];
  __syncthreads();  // reads of T and Y are done
  fa[t] = om * (sigma * eu - dn);
  fb[t] = -om * eu * sgn / h;
  __syncthreads();
  double rv = 0.0, rg = 0.0;
  if constexpr (D == 3) {
    double ra = 0.0, rb = 0.0;  // upper axis: (qb, jc)
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      ra += sG[0][q * N1 + tc] * fa[tb + N1 * q];
      rb += sG[0][q * N1 + tc] * fb[tb + N1 * q];
    }
    sY[le][0][t] = ra;
    sY[le][1][t] = rb;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      rv += sG[0][q * N1 + tb] * sY[le][0][q + N1 * tc];
      rg += sG[0][q * N1 + tb] * sY[le][1][q + N1 * tc];
    }
  } else {
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      rv += sG[0][q * N1 + tb] * fa[q];
      rg += sG[0][q * N1 + tb] * fb[q];
    }
  }
  if (act) {
    fbuf[(int64_t)f * 2 * NP + t] = (T)rv;
    fbuf[(int64_t)f * 2 * NP + NP + t] = (T)rg;
  }
}

// Diagonal correction, one thread per (face, local DoF): the default diagonal holds the
// surrogate-face term with psi_i(xi_q) (full extension); add
//   sum_q w_q (E_m psi_i - psi_i(xi_q)) (sigma_Gam psi_i(x~_q) - dn psi_i(x~_q)).
template <typename T, int D, int N1>
__global__ __launch_bounds__(kTaylorThreads) void diag_taylor_kernel(
    int n_faces, int disc_dg, int m, const int32_t *__restrict__ face_cell, const int32_t *__restrict__ face_code,
    const double *__restrict__ face_xi, const int32_t *__restrict__ runs, T *__restrict__ diag, TaylorTab tt,
    double h, double sigma) {
  constexpr int NP = D == 3 ? N1 * N1 : N1, NB = NP * N1, P = N1 - 1;
  const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (gid >= (int64_t)n_faces * NB) return;
  const int f = (int)(gid / NB), i = (int)(gid % NB);
  const int cell = face_cell[f], code = face_code[f], a = code >> 1, s = code & 1;
  const int ik[3] = {i % N1, (i / N1) % N1, D == 3 ? i / (N1 * N1) : 0};
  const double sgn = s ? 1.0 : -1.0, ds = s ? tt.D1[ik[a]] : tt.D0[ik[a]];
  double val = 0.0;
  for (int q = 0; q < NP; ++q) {
    double x0[D];
    surrogate_point<D, N1>(tt, a, s, q, x0);
    double c[D][N1];
    double full = 1.0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const double xq = face_xi[((int64_t)f * NP + q) * D + k];
      taylor_terms<N1>(tt, ik[k], x0[k], xq - x0[k], c[k]);
      // psi_i(xi_q) in product form, as the default diagonal forms it
      double l = tt.cinv[ik[k]];
#pragma unroll
      for (int j = 0; j < N1; ++j)
        if (j != ik[k]) l *= xq - tt.z[j];
      full *= l;
    }
    double em = 0.0;
#pragma unroll
    for (int j0 = 0; j0 < N1; ++j0)
#pragma unroll
      for (int j1 = 0; j1 < N1; ++j1) {
        if constexpr (D == 3) {
#pragma unroll
          for (int j2 = 0; j2 < N1; ++j2)
            if (j0 + j1 + j2 <= m) em += c[0][j0] * c[1][j1] * c[2][j2];
        } else {
          if (j0 + j1 <= m) em += c[0][j0] * c[1][j1];
        }
      }
    double tang = 1.0, om = 1.0;
    int qq = q;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (k == a) continue;
      tang *= tt.N[(qq % N1) * N1 + ik[k]];
      om *= tt.w[qq % N1] * h;
      qq /= N1;
    }
    const double vt = (ik[a] == s * P) ? tang : 0.0;
    const double dn = sgn / h * ds * tang;
    val += om * (em - full) * (sigma * vt - dn);
  }
  unsafeAtomicAdd(diag + local_dof<D, N1>(disc_dg, runs, cell, i), (T)val);
}

template <typename T, int D, int N1>
hipError_t taylor_faces(const sbm_ctx *c, const T *u, T *fbuf, hipStream_t s) {
  const int nf = (int)c->n_sbm;
  if (nf == 0) return hipSuccess;
  // one thread per (face point, slab) in the first phase (at least one wavefront)
  constexpr int NW = (D == 3 ? N1 * N1 : N1) * taylor_slabs<D, N1>();
  constexpr int NT = NW < 64 ? 64 : (NW > kTaylorThreads ? kTaylorThreads : (NW + 63) / 64 * 64);
  // orders up to 2 by sum factorisation (M = 1 or 2), the others point by point
  constexpr int EPB = low_faces_per_block<D, N1>();
  const dim3 grid((unsigned)((nf + EPB - 1) / EPB)), block(EPB * (D == 3 ? N1 * N1 : N1));
  if (c->taylor_m <= 1)
    hipLaunchKernelGGL((sbm_face_taylor_low_kernel<T, D, N1, 1>), grid, block, 0, s, nf, c->disc == SBM_DG, c->taylor_m,
                       c->d_face_cell, c->d_face_code, c->d_face_xi, c->d_face_runs, u, fbuf,
                       make_taylor_low_tab<N1, 1>(c->rules), c->h, c->sigma_gamma);
  else if (c->taylor_m == 2)
    hipLaunchKernelGGL((sbm_face_taylor_low_kernel<T, D, N1, 2>), grid, block, 0, s, nf, c->disc == SBM_DG, c->taylor_m,
                       c->d_face_cell, c->d_face_code, c->d_face_xi, c->d_face_runs, u, fbuf,
                       make_taylor_low_tab<N1, 2>(c->rules), c->h, c->sigma_gamma);
  else
    hipLaunchKernelGGL((sbm_face_taylor_kernel<T, D, N1>), dim3(nf), dim3(NT), 0, s, nf, c->disc == SBM_DG,
                       c->taylor_m, c->d_face_cell, c->d_face_code, c->d_face_xi, c->d_runs, u, fbuf,
                       make_taylor_tab(c->rules), c->h, c->sigma_gamma);
  return hipGetLastError();
}

template <typename T, int D, int N1>
hipError_t taylor_diag(const sbm_ctx *c, T *diag, hipStream_t s) {
  constexpr int NB = (D == 3 ? N1 * N1 : N1) * N1;
  const int64_t nt = c->n_sbm * (int64_t)NB;
  if (nt == 0) return hipSuccess;
  hipLaunchKernelGGL((diag_taylor_kernel<T, D, N1>), dim3((unsigned)((nt + kTaylorThreads - 1) / kTaylorThreads)),
                     dim3(kTaylorThreads), 0, s, (int)c->n_sbm, c->disc == SBM_DG, c->taylor_m, c->d_face_cell,
                     c->d_face_code, c->d_face_xi, c->d_runs, diag, make_taylor_tab(c->rules), c->h, c->sigma_gamma);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t taylor_dispatch(const sbm_ctx *c, const T *u, T *v, T *diag, hipStream_t s) {
  switch (c->p) {
#define SBM_TAYLOR_CASE(P)                                                                   \
  case P:                                                                                    \
    return diag ? taylor_diag<T, D, P + 1>(c, diag, s) : taylor_faces<T, D, P + 1>(c, u, v, s);
    SBM_TAYLOR_CASE(1)
    SBM_TAYLOR_CASE(2)
    SBM_TAYLOR_CASE(3)
    SBM_TAYLOR_CASE(4)
    SBM_TAYLOR_CASE(5)
    SBM_TAYLOR_CASE(6)
    SBM_TAYLOR_CASE(7)
    SBM_TAYLOR_CASE(8)
#undef SBM_TAYLOR_CASE
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t taylor_run(const sbm_ctx *c, const void *u, void *v, void *diag, hipStream_t s) {
  return c->dim == 3 ? taylor_dispatch<T, 3>(c, (const T *)u, (T *)v, (T *)diag, s)
                     : taylor_dispatch<T, 2>(c, (const T *)u, (T *)v, (T *)diag, s);
}

}  // namespace

hipError_t launch_operator(const sbm_ctx *c, const void *u, void *v, int prec, int parts, hipStream_t s,
                           const Scratch *scr) {
  if (c->taylor_m < 0 || !(parts & SBM_PART_SBM_FACES)) return launch_apply(c, u, v, prec, parts, s, scr);
  // the truncated surrogate-face term leaves (Rv, Rg) per face node in the face-result scratch;
  // the cell launches then take them as computed face results (SBM_PART_REUSE_FACES) and add the
  // rows in their fixed order
  void *fbuf = (scr && scr->fbuf) ? scr->fbuf : c->d_fbuf;
  if (c->n_sbm > 0) {
    const hipError_t e = prec == SBM_F64 ? taylor_run<double>(c, u, fbuf, nullptr, s)
                                         : taylor_run<float>(c, u, fbuf, nullptr, s);
    if (e != hipSuccess) return e;
  }
  return launch_apply(c, u, v, prec, parts | SBM_PART_REUSE_FACES, s, scr);
}

hipError_t launch_taylor_faces(const sbm_ctx *c, const void *u, void *fbuf, int prec, hipStream_t s) {
  if (c->n_sbm == 0) return hipSuccess;
  return prec == SBM_F64 ? taylor_run<double>(c, u, fbuf, nullptr, s) : taylor_run<float>(c, u, fbuf, nullptr, s);
}

hipError_t launch_operator_diagonal(const sbm_ctx *c, void *diag, int prec, hipStream_t s) {
  hipError_t e = launch_diagonal(c, diag, prec, s);
  if (e != hipSuccess || c->taylor_m < 0) return e;
  return prec == SBM_F64 ? taylor_run<double>(c, nullptr, nullptr, diag, s)
                         : taylor_run<float>(c, nullptr, nullptr, diag, s);
}

}  // namespace sbm
