// Planar linear advection du/dt + div(beta u) = 0 on the periodic rectangle
// (section 4.1's convergence test; equation "lin_adv"), C ABI declared in
// include/dgsw.h.
//
// The discretisation is the shallow-water one with a linear flux: orthonormal
// Legendre tensor basis, (r+1)-point Gauss-Legendre volume and edge rules,
// the weak form of equation "dg_parts", the Rusanov flux of equation
// "rusanov" (for f(u) = b u it is the upwind flux) and the mass matrix
// (dx dy / 4) I.  The operator is linear, the mesh uniform, and the rules are
// exact for products of two basis functions, so the terms of the x direction
// act on the x degree alone and leave the y degree alone, and conversely: the
// host assembles six n x n matrices (n = r + 1), per direction that of the
// element and of its two neighbours, and with q_e as the matrix [b][a]
//   dq_e/dt = q_e Sx^T + q_east Ex^T + q_west Wx^T + Sy q_e + Ny q_north + Zy q_south,
// 6n multiply-adds per output mode (the dense form of length 5 n^2, five
// n^2 x n^2 matrices, took 11.7 us a stage at 160x160 r = 3 FP64).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "dgsw.h"
#include "dgsw_ctx.hpp"
#include "dgsw_tables.hpp"

using dgsw::aligned16;
using dgsw::fail;
using dgsw::hip_fail;

struct dg_adv {
  dg_adv_desc d;
  int np = 0, N = 0, E = 0;
  int64_t state_n = 0;
  size_t elem_bytes = 0;
  void *d_ops = nullptr;     // [6][np][np] in the state dtype
};

namespace {

constexpr int kSlots = 5;    // self, east, west, north, south
constexpr int kOps = 6;      // Sx, Ex, Wx, Sy, Ny, Zy

// One direction: the element's, the next and the previous neighbour's matrix
// [m][k] (output degree, input degree) of du/dt + b du/dx = 0 on elements of
// width d, with the upwind flux: volume term (2/d) b int u phi', minus the flux
// b u_upwind times phi at the two ends.
void assemble(int np, double d, double b, double *self, double *next, double *prev) {
  std::vector<double> x, w;
  dgsw::gauss_legendre(np, x, w);
  std::vector<double> P(np * np), D(np * np), Pp(np), Pm(np);
  double pv[dgsw::kMaxNP], dv[dgsw::kMaxNP];
  for (int p = 0; p < np; ++p) {
    dgsw::legendre_onb(np - 1, x[p], pv, dv);
    for (int a = 0; a < np; ++a) { P[p * np + a] = pv[a]; D[p * np + a] = dv[a]; }
  }
  dgsw::legendre_onb(np - 1, 1.0, pv, dv);
  for (int a = 0; a < np; ++a) Pp[a] = pv[a];
  dgsw::legendre_onb(np - 1, -1.0, pv, dv);
  for (int a = 0; a < np; ++a) Pm[a] = pv[a];
  const double c = 2.0 / d;
  for (int m = 0; m < np; ++m)
    for (int k = 0; k < np; ++k) {
      double vol = 0.0;
      for (int p = 0; p < np; ++p) vol += w[p] * D[p * np + m] * P[p * np + k];
      const int i = m * np + k;
      if (b >= 0.0) {
        self[i] = c * b * (vol - Pp[m] * Pp[k]);
        next[i] = 0.0;
        prev[i] = c * b * Pm[m] * Pp[k];
      } else {
        self[i] = c * b * (vol + Pm[m] * Pm[k]);
        next[i] = -c * b * Pp[m] * Pm[k];
        prev[i] = 0.0;
      }
    }
}

struct AdvArgs {
  const void *q, *q0, *qa, *qb;
  void *out;
  int nx, ny, N, combine;          // combine: 0 rhs, 1 Shu-Osher, 2 general (as the SWE stages)
  double c0, c1, ce, dt, ca, cb;
};

// The combination's operands at one value, loaded with the stage's first loads
// (a later load would be one more trip to memory), and the combination.
template <typename T>
struct AdvOperands {
  T q0, qa, qb;
};
template <typename T>
__device__ __forceinline__ AdvOperands<T> adv_operands(size_t o, const T *q0, const T *qa, const T *qb, int combine, T c0) {
  AdvOperands<T> x;
  x.q0 = combine == 2 || (combine == 1 && c0 != T(0)) ? q0[o] : T(0);
  x.qa = combine == 2 && qa ? qa[o] : x.q0;
  x.qb = combine == 2 && qb ? qb[o] : x.q0;
  return x;
}
template <typename T>
__device__ __forceinline__ T adv_combine(T acc, T qo, const AdvOperands<T> &x, int combine, T c0, T c1, T ce, T dt,
                                         T ca, T cb) {
  if (combine == 2)
    return x.q0 + dt * acc + (c1 * (qo - x.q0) + (ca * (x.qa - x.q0) + cb * (x.qb - x.q0)));
  if (combine == 1) {
    const T y = qo + dt * acc;
    return y + c0 * (x.q0 - y) + ce * y;
  }
  return acc;
}

// Workgroups are dispatched round-robin over the 8 XCDs; renumbered so that
// each XCD takes one contiguous range of rows (its L2 then holds them and their
// neighbours).
__device__ __forceinline__ int adv_block() {
  const int nb = gridDim.x, x = blockIdx.x & 7, per = nb >> 3, rem = nb & 7;
  return x * per + (x < rem ? x : rem) + (blockIdx.x >> 3);
}

// The five stencil elements of element e = j nx + i.
__device__ __forceinline__ void adv_stencil(int e, int nx, int ny, int (&nb)[kSlots]) {
  const int j = (int)((unsigned)e / (unsigned)nx), i = e - j * nx;
  nb[0] = e;
  nb[1] = i + 1 == nx ? e + 1 - nx : e + 1;
  nb[2] = i == 0 ? e - 1 + nx : e - 1;
  nb[3] = j + 1 == ny ? i : e + nx;
  nb[4] = j == 0 ? (ny - 1) * nx + i : e - nx;
}

// One lane per (element, output mode (b, a)), G = 256 / N consecutive elements
// per workgroup.  The matrices and the G elements' five stencil rows are staged
// in LDS (the rows with coalesced loads, one value per lane per slot).
template <typename T, int NP>
__global__ __launch_bounds__(256) void k_adv_stage(const T *__restrict__ ops, const T *__restrict__ q,
                                                   const T *q0, const T *qa, const T *qb, T *out, int nx, int ny,
                                                   int combine, T c0, T c1, T ce, T dt, T ca, T cb) {
  constexpr int N = NP * NP, G = 256 / N;
  // padded strides: rows of different output modes / elements start in
  // different LDS banks
  constexpr int LA = NP + 1, LQ = kSlots * N + 1;
  __shared__ T sA[kOps * NP * LA];
  __shared__ T sQ[G * LQ];
  for (int k = threadIdx.x; k < kOps * N; k += 256) sA[(k / NP) * LA + k % NP] = ops[k];
  const int64_t E = (int64_t)nx * ny;
  const int g = threadIdx.x / N, m = threadIdx.x - g * N, b = m / NP, a = m - b * NP;
  const int64_t e64 = (int64_t)adv_block() * G + g;
  const bool live = g < G && e64 < E;
  const int e = live ? (int)e64 : 0;
  const size_t o = (size_t)e * N + m;
  AdvOperands<T> x{T(0), T(0), T(0)};
  if (g < G) {
    int nb[kSlots];
    adv_stencil(e, nx, ny, nb);
    T v[kSlots];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) v[k] = q[(size_t)nb[k] * N + m];
    x = adv_operands<T>(o, q0, qa, qb, combine, c0);
#pragma unroll
    for (int k = 0; k < kSlots; ++k) sQ[g * LQ + k * N + m] = v[k];
  }
  __syncthreads();
  if (!live) return;
  const T *S = sQ + g * LQ;
  const T *rx = S + b * NP, *ry = S + a;               // row b (x degrees) and column a (y degrees)
  T acc = T(0);
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    acc += sA[(0 * NP + a) * LA + k] * rx[k];
    acc += sA[(1 * NP + a) * LA + k] * rx[N + k];
    acc += sA[(2 * NP + a) * LA + k] * rx[2 * N + k];
    acc += sA[(3 * NP + b) * LA + k] * ry[k * NP];
    acc += sA[(4 * NP + b) * LA + k] * ry[3 * N + k * NP];
    acc += sA[(5 * NP + b) * LA + k] * ry[4 * N + k * NP];
  }
  out[o] = adv_combine<T>(acc, S[m], x, combine, c0, c1, ce, dt, ca, cb);
}

// r = 3 in FP64: each of the six terms is one v_mfma_f64_4x4x4 block per
// element, four elements per wavefront (lane l: element (l / 4) % 4, entry
// (x, y) = (l / 16, l % 4) of every 4 x 4 array; A[i = y][k = x], B[k = x][j = y],
// result [x][y]).  The stencil is loaded in memory order (a wavefront's 64
// lanes read 512 contiguous bytes a slot), turned to the operand layouts
// through LDS, and so is the result.  160x160: 11.9 -> 4.5 us a stage, of which
// the launch is about half; before the XCD renumbering and with the
// combination's operands loaded after the products 5.1.
__global__ __launch_bounds__(256) void k_adv_stage_m4(const double *__restrict__ ops, const double *__restrict__ q,
                                                      const double *q0, const double *qa, const double *qb,
                                                      double *out, int nx, int ny, int combine, double c0, double c1,
                                                      double ce, double dt, double ca, double cb) {
  constexpr int LE = 24, LS = 4 * LE;                  // padded strides of an element and a slot
  __shared__ double sA[kOps * 16];
  __shared__ double sQ[4][kSlots * LS];
  if (threadIdx.x < kOps * 16) sA[threadIdx.x] = ops[threadIdx.x];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int E = nx * ny;
  const int e_raw = adv_block() * 16 + wv * 4 + (lane >> 4), m = lane & 15;
  const bool live = e_raw < E;
  const int e = live ? e_raw : E - 1;
  const size_t o = (size_t)e * 16 + m;
  double *S = sQ[wv];
  double qo;
  AdvOperands<double> op;
  {
    int nb[kSlots];
    adv_stencil(e, nx, ny, nb);
    double v[kSlots];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) v[k] = q[(size_t)nb[k] * 16 + m];
    op = adv_operands<double>(o, q0, qa, qb, combine, c0);
    qo = v[0];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) S[k * LS + (lane >> 4) * LE + m] = v[k];
  }
  __syncthreads();
  const int x = lane >> 4, y = lane & 3, at = ((lane >> 2) & 3) * LE;
  const int n = at + 4 * x + y, t = at + 4 * y + x, c = 4 * y + x;
  double acc = __builtin_amdgcn_mfma_f64_4x4x4f64(S[t], sA[c], 0.0, 0, 0, 0);
  double acy = __builtin_amdgcn_mfma_f64_4x4x4f64(sA[48 + c], S[n], 0.0, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f64_4x4x4f64(S[LS + t], sA[16 + c], acc, 0, 0, 0);
  acy = __builtin_amdgcn_mfma_f64_4x4x4f64(sA[64 + c], S[3 * LS + n], acy, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f64_4x4x4f64(S[2 * LS + t], sA[32 + c], acc, 0, 0, 0);
  acy = __builtin_amdgcn_mfma_f64_4x4x4f64(sA[80 + c], S[4 * LS + n], acy, 0, 0, 0);
  __syncthreads();
  S[n] = acc + acy;
  __syncthreads();
  if (!live) return;
  out[o] = adv_combine<double>(S[(lane >> 4) * LE + m], qo, op, combine, c0, c1, ce, dt, ca, cb);
}

template <typename T, int NP>
hipError_t launch_adv_t(const dg_adv *a, const AdvArgs &g, hipStream_t s) {
  constexpr int G = 256 / (NP * NP);
  const int64_t E = (int64_t)g.nx * g.ny;
  const dim3 grid((unsigned)((E + G - 1) / G)), block(256);
  const T *ops = static_cast<const T *>(a->d_ops), *q = static_cast<const T *>(g.q), *q0 = static_cast<const T *>(g.q0);
  const T *qa = static_cast<const T *>(g.qa), *qb = static_cast<const T *>(g.qb);
  T *out = static_cast<T *>(g.out);
  if constexpr (sizeof(T) == 8 && NP == 4)
    hipLaunchKernelGGL(k_adv_stage_m4, grid, block, 0, s, ops, q, q0, qa, qb, out, g.nx, g.ny, g.combine, g.c0, g.c1,
                       g.ce, g.dt, g.ca, g.cb);
  else
    hipLaunchKernelGGL((k_adv_stage<T, NP>), grid, block, 0, s, ops, q, q0, qa, qb, out, g.nx, g.ny, g.combine,
                       T(g.c0), T(g.c1), T(g.ce), T(g.dt), T(g.ca), T(g.cb));
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adv_d(const dg_adv *a, const AdvArgs &g, hipStream_t s) {
  switch (a->np) {
    case 1: return launch_adv_t<T, 1>(a, g, s);
    case 2: return launch_adv_t<T, 2>(a, g, s);
    case 3: return launch_adv_t<T, 3>(a, g, s);
    case 4: return launch_adv_t<T, 4>(a, g, s);
    case 5: return launch_adv_t<T, 5>(a, g, s);
    case 6: return launch_adv_t<T, 6>(a, g, s);
    case 7: return launch_adv_t<T, 7>(a, g, s);
    default: return hipErrorInvalidValue;
  }
}

int adv_stage(dg_adv *a, const void *q, const void *q0, void *out, int combine, double c0, double c1, double dt,
              const void *qa, double ca, const void *qb, double cb, hipStream_t s) {
  AdvArgs g;
  g.q = q; g.q0 = q0; g.qa = qa; g.qb = qb; g.out = out;
  g.nx = a->d.nx; g.ny = a->d.ny; g.N = a->N; g.combine = combine;
  g.c0 = c0; g.c1 = c1; g.ce = c0 + c1 - 1.0; g.dt = dt; g.ca = ca; g.cb = cb;
  hipError_t e = a->d.dtype == DG_F64 ? launch_adv_d<double>(a, g, s) : launch_adv_d<float>(a, g, s);
  if (e != hipSuccess) return hip_fail(e, "advection stage launch");
  return DG_OK;
}

}  // namespace

extern "C" {

int dg_adv_init(const dg_adv_desc *d, void *hip_stream, dg_adv **out) {
  if (!out) return fail(DG_EINVAL, "out is NULL");
  *out = nullptr;
  if (!d) return fail(DG_EINVAL, "desc is NULL");
  if (d->abi_version != DG_ABI_VERSION) return fail(DG_EINVAL, "abi_version mismatch");
  if (d->nx < 1 || d->ny < 1) return fail(DG_EINVAL, "nx and ny must be >= 1");
  if (d->order < 0) return fail(DG_EINVAL, "order must be >= 0");
  if (d->order > 6) return fail(DG_EUNSUPPORTED, "order > 6 is not supported for advection");
  if (d->reserved != 0) return fail(DG_EINVAL, "reserved must be 0");
  if (d->dtype != DG_F64 && d->dtype != DG_F32) return fail(DG_EDTYPE, "dtype must be DG_F64 or DG_F32");
  if (!(d->lx > 0.0) || !std::isfinite(d->lx) || !(d->ly > 0.0) || !std::isfinite(d->ly))
    return fail(DG_EINVAL, "lx and ly must be > 0");
  if (!std::isfinite(d->bx) || !std::isfinite(d->by)) return fail(DG_EINVAL, "beta must be finite");
  const int64_t np = d->order + 1;
  if ((int64_t)d->nx * d->ny * np * np >= (int64_t(1) << 31)) return fail(DG_EINVAL, "state exceeds 2^31 values");
  dg_adv *a = new dg_adv();
  a->d = *d;
  a->np = (int)np;
  a->N = (int)(np * np);
  a->E = d->nx * d->ny;
  a->state_n = (int64_t)a->E * a->N;
  a->elem_bytes = d->dtype == DG_F64 ? 8 : 4;
  std::vector<double> A((size_t)kOps * a->N);
  assemble(a->np, d->lx / d->nx, d->bx, &A[0], &A[a->N], &A[2 * a->N]);
  assemble(a->np, d->ly / d->ny, d->by, &A[3 * a->N], &A[4 * a->N], &A[5 * a->N]);
  std::vector<unsigned char> h(A.size() * a->elem_bytes);
  if (d->dtype == DG_F64) {
    std::memcpy(h.data(), A.data(), h.size());
  } else {
    for (size_t k = 0; k < A.size(); ++k) {
      const float f = (float)A[k];
      std::memcpy(h.data() + 4 * k, &f, 4);
    }
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  hipError_t e;
  if ((e = hipMalloc(&a->d_ops, h.size())) != hipSuccess) {
    delete a;
    return fail(DG_ENOMEM, "hipMalloc of the advection operator");
  }
  if ((e = hipMemcpyAsync(a->d_ops, h.data(), h.size(), hipMemcpyHostToDevice, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess) {
    (void)hipFree(a->d_ops);
    delete a;
    return hip_fail(e, "upload of the advection operator");
  }
  *out = a;
  return DG_OK;
}

int dg_adv_free(dg_adv *a) {
  if (!a) return DG_OK;
  if (a->d_ops) (void)hipFree(a->d_ops);
  delete a;
  return DG_OK;
}

int dg_adv_state_size(const dg_adv *a, int64_t *n_values) {
  if (!a || !n_values) return fail(DG_EINVAL, "NULL argument");
  *n_values = a->state_n;
  return DG_OK;
}

int dg_adv_rhs(dg_adv *a, const void *q, void *dqdt, void *hip_stream) {
  if (!a || !q || !dqdt) return fail(DG_EINVAL, "NULL argument");
  if (!aligned16(q) || !aligned16(dqdt)) return fail(DG_EINVAL, "state pointers must be 16-byte aligned");
  const size_t bytes = a->state_n * a->elem_bytes;
  const char *x = static_cast<const char *>(q), *y = static_cast<const char *>(dqdt);
  if (x < y + bytes && y < x + bytes) return fail(DG_EINVAL, "q and dqdt overlap");
  return adv_stage(a, q, nullptr, dqdt, 0, 0.0, 1.0, 0.0, nullptr, 0.0, nullptr, 0.0,
                   static_cast<hipStream_t>(hip_stream));
}

int dg_adv_rk_step(dg_adv *a, void *q, void *work, double dt, int32_t scheme, int32_t nsteps, void *hip_stream) {
  if (!a || !q || !work) return fail(DG_EINVAL, "NULL argument");
  if (!aligned16(q) || !aligned16(work)) return fail(DG_EINVAL, "state pointers must be 16-byte aligned");
  if (nsteps < 0 || !std::isfinite(dt)) return fail(DG_EINVAL, "bad nsteps or dt");
  int nwork;
  switch (scheme) {
    case DG_SSP_RK1: nwork = 1; break;
    case DG_SSP_RK2:
    case DG_SSP_RK3: nwork = 2; break;
    case DG_RK4: nwork = 3; break;
    default: return fail(DG_EINVAL, "unknown scheme");
  }
  const size_t bytes = a->state_n * a->elem_bytes;
  {
    const char *x = static_cast<const char *>(q), *y = static_cast<const char *>(work);
    if (x < y + nwork * bytes && y < x + bytes) return fail(DG_EINVAL, "q and work overlap");
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  char *w0 = static_cast<char *>(work), *w1 = w0 + bytes, *w2 = w1 + bytes;
  int rc;
  for (int n = 0; n < nsteps; ++n) {
    switch (scheme) {
      case DG_SSP_RK1: {
        if ((rc = adv_stage(a, q, nullptr, w0, 1, 0.0, 1.0, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        hipError_t e = hipMemcpyAsync(q, w0, bytes, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "RK1 copy-back");
        break;
      }
      case DG_SSP_RK2:
        if ((rc = adv_stage(a, q, nullptr, w0, 1, 0.0, 1.0, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w0, q, q, 1, 0.5, 0.5, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        break;
      case DG_SSP_RK3:
        if ((rc = adv_stage(a, q, nullptr, w0, 1, 0.0, 1.0, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w0, q, w1, 1, 0.75, 0.25, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w1, q, q, 1, 1.0 / 3.0, 2.0 / 3.0, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        break;
      case DG_RK4:
        if ((rc = adv_stage(a, q, nullptr, w0, 1, 0.0, 1.0, 0.5 * dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w0, q, w1, 2, 1.0, 0.0, 0.5 * dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w1, q, w2, 2, 1.0, 0.0, dt, nullptr, 0, nullptr, 0, s)) != DG_OK) return rc;
        if ((rc = adv_stage(a, w2, q, q, 2, 0.0, 1.0 / 3.0, dt / 6.0, w0, 1.0 / 3.0, w1, 2.0 / 3.0, s)) != DG_OK)
          return rc;
        break;
    }
  }
  return DG_OK;
}

}  // extern "C"
