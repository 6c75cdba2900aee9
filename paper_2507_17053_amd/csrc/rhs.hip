// Right-hand side of Eq. (1), on the device and, for the smallest operators, on the host:
//   b_i = int f psi_i - int_{Gam~} (dpsi_i/dn~) g + int_{Gam~} sigma g psi_i
// from f at the cells' Gauss points and g at the true-boundary points (host arrays).
//
// Every integral is a tensor-product quadrature, so the transposed interpolation to the basis is
// done axis by axis (N^T along each axis in turn):
//   cell:  loc_i = sum_q psi_i(g_q) W_q h^d f(x_q)
//   face:  loc_i += c(i_a) T(i_t), T = sum_q psi_t(g_q) omega_q g(x_q) over the tangential axes,
//          c(i_a) = sigma [i_a = s p] - sgn / h l'_{i_a}(s)   (sigma g v - g dv/dn~)
// A cell adds its surrogate faces' vectors (in face order) to its own before its one addition to b.
// Cells of one parity of their mesh coordinates share no DoF, so a CG right-hand side is 2^d
// launches, one per parity, each with plain additions: every DoF sums its cells in an order fixed
// by the setup (by chunk, then parity), with no atomics and no scratch beyond the data.
//
// What bounds it: the copy of f from the caller's memory (8 (p+1)^d bytes per cell, 28 GB/s from
// ordinary host memory) and, for CG, 2^d launches of which each covers one cell in 2^d.  The same sums
// on 16 host threads took 2.76 ms for 40^3 Q4, 0.36 ms here (0.08 ms of it kernels).  f goes to the
// device in chunks of at most 64 MB, so that the scratch stays small beside the operator at any size.
// An operator of few cells is assembled on the calling thread (host_work).
#include <algorithm>
#include <new>
#include <vector>

#include "sbm_internal.h"

namespace sbm {
namespace {

constexpr size_t kChunkBytes = (size_t)64 << 20;  // of f on the device at a time

template <int N1>
struct RhsTab {
  double R[N1 * N1];  // R[i N1 + q] = l_i(g_q) w_q
  double N[N1 * N1];  // N[q N1 + i] = l_i(g_q)
  double D0[N1], D1[N1], w[N1];
};

// The surrogate faces of each cell (faces are listed by cell, then code): first face and mask of
// the codes 2 axis + side.  cf is zero before.
__global__ __launch_bounds__(256) void rhs_faces_kernel(int64_t nf, const int32_t *__restrict__ faces,
                                                        int2 *__restrict__ cf) {
  const int64_t f = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (f >= nf) return;
  const int32_t r = faces[3 * f];
  if (f > 0 && faces[3 * (f - 1)] == r) return;
  int mask = 0;
  for (int64_t k = f; k < nf && k < f + 6 && faces[3 * k] == r; ++k)
    mask |= 1 << (2 * faces[3 * k + 1] + faces[3 * k + 2]);
  cf[r] = make_int2((int)f, mask);
}

template <int D, int N1>
struct RhsShape {
  static constexpr int NP = D == 3 ? N1 * N1 : N1, NB = NP * N1, EPB = 256 / NP;
};

// NP threads per cell, EPB cells per workgroup.  Cells r0 .. r0 + n of the mesh; f: their block.
// color: -1 (DG: every cell, b stored) or the parity of the launch (CG, added to b).
template <int D, int N1>
__global__ __launch_bounds__(256) void rhs_cells_kernel(int n, int64_t r0, int color,
                                                        const int32_t *__restrict__ cells,
                                                        const int2 *__restrict__ cf, const double *__restrict__ f,
                                                        const double *__restrict__ g,
                                                        const int32_t *__restrict__ runs, double *__restrict__ b,
                                                        RhsTab<N1> tab, double h, double sigma) {
  using S = RhsShape<D, N1>;
  constexpr int NP = S::NP, NB = S::NB, EPB = S::EPB, P = N1 - 1;
  __shared__ double tile[EPB * NB];
  __shared__ double face[2][EPB * NP];
  const int le = threadIdx.x / NP, t = threadIdx.x - le * NP;
  const int c = blockIdx.x * EPB + le;
  const int64_t rank = r0 + c;
  bool mine = c < n;
  if (mine && color >= 0) {
    int par = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) par |= (cells[rank * D + k] & 1) << k;
    mine = par == color;
  }
  if (!__syncthreads_or(mine)) return;
  double *const A = tile + le * NB;
  const int t0 = D == 3 ? t % N1 : t, t1 = D == 3 ? t / N1 : 0;
  auto sweep = [&](const double (&x)[N1], double (&y)[N1]) {  // N^T W along one axis
#pragma unroll
    for (int i = 0; i < N1; ++i) {
      double a = 0.0;
#pragma unroll
      for (int q = 0; q < N1; ++q) a += tab.R[i * N1 + q] * x[q];
      y[i] = a;
    }
  };
  double x[N1], out[N1];
#pragma unroll
  for (int k = 0; k < N1; ++k) x[k] = mine ? f[(int64_t)c * NB + t + NP * k] : 0.0;
  sweep(x, out);
#pragma unroll
  for (int i = 0; i < N1; ++i) A[t + NP * i] = out[i];
  __syncthreads();
  if constexpr (D == 3) {
#pragma unroll
    for (int k = 0; k < N1; ++k) x[k] = A[t0 + N1 * k + NP * t1];
    sweep(x, out);
#pragma unroll
    for (int i = 0; i < N1; ++i) A[t0 + N1 * i + NP * t1] = out[i];
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < N1; ++k) x[k] = A[k + N1 * t];
  sweep(x, out);  // the thread's x-run t of the cell
  const double hd = D == 3 ? h * h * h : h * h;
#pragma unroll
  for (int i = 0; i < N1; ++i) out[i] *= hd;
  // surrogate faces, in code order
  const int2 mf = mine ? cf[rank] : make_int2(0, 0);
  double *const G = face[0] + le * NP, *const H = face[1] + le * NP;
  const double om = D == 3 ? tab.w[t0] * tab.w[t1] * h * h : tab.w[t0] * h;
#pragma unroll
  for (int code = 0; code < 2 * D; ++code) {
    const bool has = (mf.y >> code) & 1;
    if (!__syncthreads_or(has)) continue;
    const int64_t fi = mf.x + __popc(mf.y & ((1 << code) - 1));
    G[t] = has ? om * g[fi * NP + t] : 0.0;
    __syncthreads();
    const double *T;
    if constexpr (D == 3) {
      double a = 0.0;
#pragma unroll
      for (int q = 0; q < N1; ++q) a += tab.N[q * N1 + t0] * G[q + N1 * t1];
      H[t] = a;
      __syncthreads();
      a = 0.0;
#pragma unroll
      for (int q = 0; q < N1; ++q) a += tab.N[q * N1 + t1] * H[t0 + N1 * q];
      G[t] = a;
      T = G;
    } else {
      double a = 0.0;
#pragma unroll
      for (int q = 0; q < N1; ++q) a += tab.N[q * N1 + t] * G[q];
      H[t] = a;
      T = H;
    }
    __syncthreads();
    if (has) {
      const int a = code >> 1, s = code & 1;
      const double sg = s ? 1.0 : -1.0;
      auto row = [&](int ia) {  // c(ia)
        return (ia == s * P ? sigma : 0.0) - sg / h * (s ? tab.D1[ia] : tab.D0[ia]);
      };
      if (a == 0) {
        const double v = T[t];
#pragma unroll
        for (int i = 0; i < N1; ++i) out[i] += row(i) * v;
      } else {
        const int ia = a == 1 ? t0 : t1;  // the run's place along the normal
        double ci = 0.0;
#pragma unroll
        for (int i = 0; i < N1; ++i) ci = i == ia ? row(i) : ci;
#pragma unroll
        for (int i = 0; i < N1; ++i) out[i] += ci * T[D == 3 ? i + N1 * (a == 1 ? t1 : t0) : i];
      }
    }
  }
  if (!mine) return;
  if (color < 0) {
#pragma unroll
    for (int i = 0; i < N1; ++i) b[rank * NB + N1 * t + i] = out[i];
  } else {
    double *const to = b + runs[rank * NP + t];
#pragma unroll
    for (int i = 0; i < N1; ++i) to[i] += out[i];
  }
}

template <int D, int N1>
hipError_t rhs_chunk(const sbm_ctx *c, int n, int64_t r0, const int32_t *cells, const int2 *cf, const double *f,
                     const double *g, double *b, hipStream_t s) {
  using S = RhsShape<D, N1>;
  const Rules1D &r = c->rules;
  RhsTab<N1> tab;
  for (int i = 0; i < N1; ++i) {
    for (int q = 0; q < N1; ++q) {
      tab.R[i * N1 + q] = r.N[q * N1 + i] * r.w[q];
      tab.N[q * N1 + i] = r.N[q * N1 + i];
    }
    tab.D0[i] = r.D0[i];
    tab.D1[i] = r.D1[i];
    tab.w[i] = r.w[i];
  }
  const dim3 grid((unsigned)((n + S::EPB - 1) / S::EPB)), block(S::EPB * S::NP);
  const bool cg = c->disc == SBM_CG;
  for (int color = cg ? 0 : -1; color < (cg ? 1 << D : 0); ++color)
    hipLaunchKernelGGL((rhs_cells_kernel<D, N1>), grid, block, 0, s, n, r0, color, cells, cf, f, g, c->d_runs, b, tab,
                       c->h, c->sigma_gamma);
  return hipGetLastError();
}

template <int D>
hipError_t rhs_degree(const sbm_ctx *c, int n, int64_t r0, const int32_t *cells, const int2 *cf, const double *f,
                      const double *g, double *b, hipStream_t s) {
  switch (c->p) {
    case 1: return rhs_chunk<D, 2>(c, n, r0, cells, cf, f, g, b, s);
    case 2: return rhs_chunk<D, 3>(c, n, r0, cells, cf, f, g, b, s);
    case 3: return rhs_chunk<D, 4>(c, n, r0, cells, cf, f, g, b, s);
    case 4: return rhs_chunk<D, 5>(c, n, r0, cells, cf, f, g, b, s);
    case 5: return rhs_chunk<D, 6>(c, n, r0, cells, cf, f, g, b, s);
    case 6: return rhs_chunk<D, 7>(c, n, r0, cells, cf, f, g, b, s);
    case 7: return rhs_chunk<D, 8>(c, n, r0, cells, cf, f, g, b, s);
    case 8: return rhs_chunk<D, 9>(c, n, r0, cells, cf, f, g, b, s);
  }
  return hipErrorInvalidValue;
}

// Everything of one call on stream s; scratch is the call's device block.
hipError_t rhs_on(const sbm_ctx *c, const double *f_qp, const double *g_bp, double *b, char *scratch,
                  const size_t (&off)[5], int64_t chunk, hipStream_t s) {
  const int64_t nc = c->n_cells, nf = c->n_sbm, nb = c->nb, d = c->dim;
  int32_t *cells = (int32_t *)(scratch + off[0]), *faces = (int32_t *)(scratch + off[1]);
  int2 *cf = (int2 *)(scratch + off[2]);
  double *g = (double *)(scratch + off[3]), *f = (double *)(scratch + off[4]);
  hipError_t e = vec_fill(cf, nc, 0.0, SBM_F64, s);  // (an all-zero double is an all-zero int2)
  if (e == hipSuccess && c->disc == SBM_CG) {
    e = vec_fill(b, c->n_dofs, 0.0, SBM_F64, s);
    if (e == hipSuccess) e = hipMemcpyAsync(cells, c->cells.data(), sizeof(int32_t) * nc * d, hipMemcpyHostToDevice, s);
  }
  if (e == hipSuccess && nf > 0) {
    e = hipMemcpyAsync(faces, c->faces.data(), sizeof(int32_t) * 3 * nf, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(g, g_bp, sizeof(double) * nf * c->nq_face, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rhs_faces_kernel, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s, nf, faces, cf);
    e = hipGetLastError();
  }
  for (int64_t r0 = 0; e == hipSuccess && r0 < nc; r0 += chunk) {
    const int64_t n = std::min(chunk, nc - r0);
    e = hipMemcpyAsync(f, f_qp + r0 * nb, sizeof(double) * n * nb, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = d == 3 ? rhs_degree<3>(c, (int)n, r0, cells, cf, f, g, b, s) : rhs_degree<2>(c, (int)n, r0, cells, cf, f, g, b, s);
  }
  return e;
}

// out = N^T in along one axis of a tensor of n1 points per axis (first axis fastest)
void contract(const Rules1D &R, int n1, const double *in, double *out, int dims, int axis) {
  int st = 1, outer = 1;
  for (int m = 0; m < axis; ++m) st *= n1;
  for (int m = axis + 1; m < dims; ++m) outer *= n1;
  for (int o = 0; o < outer; ++o) {
    const double *src = in + (size_t)o * n1 * st;
    double *dst = out + (size_t)o * n1 * st;
    for (int i = 0; i < n1; ++i)
      for (int l = 0; l < st; ++l) {
        double acc = 0.0;
        for (int q = 0; q < n1; ++q) acc += R.N[q * n1 + i] * src[q * st + l];
        dst[i * st + l] = acc;
      }
  }
}

// All of it on one host thread: the cells in rank order, then the faces in face order.
void rhs_host(const sbm_ctx *h, const double *f_qp, const double *g_bp, double *b) {
  const int d = h->dim, n1 = h->n1, nb = h->nb, np = h->nq_face, P = h->p;
  const Rules1D &R = h->rules;
  std::vector<double> A(nb), B(nb);
  double *src = A.data(), *dst = B.data();
  std::vector<double> w(nb), wf(np);  // quadrature weights of a cell and of a face
  for (int q = 0; q < nb; ++q) {
    const int qk[3] = {q % n1, (q / n1) % n1, q / (n1 * n1)};
    w[q] = 1.0;
    for (int m = 0; m < d; ++m) w[q] *= R.w[qk[m]] * h->h;
    if (q < np) {
      wf[q] = 1.0;
      for (int m = 0; m < d - 1; ++m) wf[q] *= R.w[qk[m]] * h->h;
    }
  }
  std::fill(b, b + h->n_dofs, 0.0);
  // local entry i of cell r, i = n1 t + k
  auto run = [&](int64_t r, int t) { return b + (h->disc == SBM_CG ? (int64_t)h->runs[r * np + t] : r * nb + n1 * t); };
  for (int64_t r = 0; r < h->n_cells; ++r) {
    for (int q = 0; q < nb; ++q) src[q] = f_qp[r * nb + q] * w[q];
    for (int m = 0; m < d; ++m) {
      contract(R, n1, src, dst, d, m);
      std::swap(src, dst);
    }
    for (int t = 0; t < np; ++t) {
      double *to = run(r, t);
      for (int k = 0; k < n1; ++k) to[k] += src[n1 * t + k];
    }
  }
  for (int64_t f = 0; f < h->n_sbm; ++f) {
    const int32_t *fc = &h->faces[3 * f];
    const int a = fc[1], s = fc[2];
    const double *Ds = s ? R.D1.data() : R.D0.data();
    const double sgn = s ? 1.0 : -1.0;
    for (int q = 0; q < np; ++q) src[q] = wf[q] * g_bp[f * np + q];
    for (int m = 0; m < d - 1; ++m) {
      contract(R, n1, src, dst, d - 1, m);
      std::swap(src, dst);
    }
    auto row = [&](int ia) { return (ia == s * P ? h->sigma_gamma : 0.0) - sgn / h->h * Ds[ia]; };
    for (int t = 0; t < np; ++t) {
      const int t0 = t % n1, t1 = t / n1;
      double *to = run(fc[0], t);
      for (int k = 0; k < n1; ++k)
        to[k] += a == 0 ? row(k) * src[t] : (a == 1 ? row(t0) * src[d == 3 ? k + n1 * t1 : k] : row(t1) * src[k + n1 * t0]);
    }
  }
}

sbm_status by_host(const sbm_ctx *h, const double *f_qp, const double *g_bp, double *b, hipStream_t s) {
  try {
    std::vector<double> bh(h->n_dofs);
    rhs_host(h, f_qp, g_bp, bh.data());
    const hipError_t e = hipMemcpyAsync(b, bh.data(), sizeof(double) * bh.size(), hipMemcpyHostToDevice, s);
    SBM_HIP_CHECK(hipStreamSynchronize(s));
    SBM_HIP_CHECK(e);
  } catch (const std::bad_alloc &) {
    set_error("sbm_rhs: out of host memory");
    return SBM_ENOMEM;
  }
  return SBM_OK;
}

// On the device, f in pieces of at most `chunk` cells.
sbm_status by_device(const sbm_ctx *h, const double *f_qp, const double *g_bp, double *b, int64_t chunk, hipStream_t s) {
  const int64_t nc = h->n_cells, nf = h->n_sbm;
  const size_t need[5] = {sizeof(int32_t) * nc * h->dim, sizeof(int32_t) * 3 * nf, sizeof(int2) * nc,
                          sizeof(double) * nf * h->nq_face, sizeof(double) * chunk * h->nb};
  size_t off[5], bytes = 0;
  for (int k = 0; k < 5; ++k) {
    off[k] = bytes;
    bytes += (need[k] + 255) / 256 * 256;
  }
  void *scratch = nullptr;
  const hipError_t ea = dev_alloc(&scratch, bytes);
  if (ea != hipSuccess) {
    (void)hipGetLastError();
    set_error(std::string("sbm_rhs: scratch allocation failed: ") + hipGetErrorString(ea));
    return ea == hipErrorOutOfMemory ? SBM_ENOMEM : SBM_EHIP;
  }
  const hipError_t e = rhs_on(h, f_qp, g_bp, b, (char *)scratch, off, chunk, s);
  const hipError_t es = hipStreamSynchronize(s);  // the scratch is free, and b ready
  dev_free(scratch);
  SBM_HIP_CHECK(e);
  SBM_HIP_CHECK(es);
  return SBM_OK;
}

// Multiply-adds of the host form, with 50 (d - 1) more per cell for its loops: it takes 20 us and
// 0.23 us per thousand.  The device form takes 70 us and more for CG (its launches and copies), 33 us and
// more for DG.  Host / device in us at sizes about the lines drawn here: CG 2D Q1, 5,771 cells (384 k)
// 105 / 95, 3D Q3, 112 cells (130 k) 60 / 149, 2D Q2, 1,399 cells (149 k) 60 / 84; DG 2D Q1, 1,399 cells
// (94 k) 39 / 48, 3D Q6, 7 cells (82 k) 41 / 55, 3D Q3, 7 cells (12 k) 24 / 37.
int64_t host_work(const sbm_ctx *h) {
  return h->n_cells * (h->nb * h->dim * h->n1 + 50 * (h->dim - 1)) +
         h->n_sbm * (h->nq_face * (h->dim - 1) * h->n1 + h->nb);
}
constexpr int64_t kHostWork[2] = {250000, 80000};  // SBM_CG, SBM_DG

}  // namespace
}  // namespace sbm

extern "C" sbm_status sbm_rhs_form(sbm_handle h, const double *f_qp, const double *g_bp, double *b, int form,
                                   int64_t cells, void *stream) {
  using namespace sbm;
  if (!h || !f_qp || !b || (h->n_sbm > 0 && !g_bp) || h->host_only || cells < 0 || form < SBM_RHS_AUTO ||
      form > SBM_RHS_DEVICE) {
    set_error("sbm_rhs: NULL argument or host-only handle");
    return SBM_EINVAL;
  }
  const hipStream_t s = (hipStream_t)stream;
  if (h->n_cells == 0) {
    SBM_HIP_CHECK(hipStreamSynchronize(s));
    return SBM_OK;
  }
  if (form == SBM_RHS_HOST || (form == SBM_RHS_AUTO && host_work(h) <= kHostWork[h->disc == SBM_DG]))
    return by_host(h, f_qp, g_bp, b, s);
  const int64_t most = std::max<int64_t>(1, (int64_t)(kChunkBytes / (sizeof(double) * h->nb)));
  const sbm_status st = by_device(h, f_qp, g_bp, b, std::min(h->n_cells, cells > 0 ? std::min(cells, most) : most), s);
  // (no room on the device beside its other contents: the host form needs none)
  return st == SBM_ENOMEM && form == SBM_RHS_AUTO ? by_host(h, f_qp, g_bp, b, s) : st;
}

extern "C" sbm_status sbm_rhs(sbm_handle h, const double *f_qp, const double *g_bp, double *b, void *stream) {
  return sbm_rhs_form(h, f_qp, g_bp, b, SBM_RHS_AUTO, 0, stream);
}
