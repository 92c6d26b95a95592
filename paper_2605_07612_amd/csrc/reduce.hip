// FP64 reductions and flux fixing: CFL time step, step finalisation,
// conserved totals, and the flux correction at refinement boundaries
// (Sec. 2.7).
#include "device_common.h"
#include "foap4_internal.h"
#include "stage_common.h"

#include <mutex>

namespace f4 {

// Scalar advection (Sec. 3.4): the fastest wave along d is |v_d| in every
// cell, so the CFL limit is sum_d |v_d| / dx (the definition's operation
// order); a non-finite rho marks the state bad.
template <int NDIM>
__device__ __forceinline__ double inv_dt_adv(const MeshDev &M, double rho, double dx, bool &bad) {
#pragma clang fp contract(off)
  double s = 0.0;
#pragma unroll
  for (int d = 0; d < NDIM; d++) s += fabs(M.vel[d]) / dx;
  bad |= !isfinite(rho);
  return s;
}

__device__ __forceinline__ void wave_flush(double *scal, double vmax, bool bad) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vmax = fmax(vmax, __shfl_xor(vmax, o));
  const bool anybad = __ballot(bad) != 0;
  if ((threadIdx.x & 63) == 0) {
    if (vmax > 0.0) atomic_max_pos_if_larger(&scal[kMaxInv], vmax);
    if (anybad) atomic_max_pos(&scal[kBad], 1.0);
  }
}

// CFL limit of every interior cell of the current state (one workgroup per block)
template <typename T, int NDIM, int NV>
__global__ __launch_bounds__(256) void dt_full_kernel(const MeshDev *__restrict__ Mp) {
  const MeshDev &M = *Mp;
  const int64_t b = blockIdx.x;
  const int N = M.N, g = M.g, P = N + 2 * g;
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  const T *u = (const T *)M.s[M.cur] + b * sv * NV;
  const double dx = ldexp(M.dx0, -M.level[b]);
  const int cells = (NDIM == 3) ? N * N * N : N * N;
  double vmax = 0.0;
  bool bad = false;
  for (int c = threadIdx.x; c < cells; c += blockDim.x) {
    const int i = c % N, j = (c / N) % N, k = (NDIM == 3) ? c / (N * N) : 0;
    const int64_t o = cell_off<NDIM>(i, j, k, N, g);
    double U[NV];
#pragma unroll
    for (int v = 0; v < NV; v++) U[v] = (double)u[v * sv + o];
    if constexpr (NV == 1) vmax = fmax(vmax, inv_dt_adv<NDIM>(M, U[0], dx, bad));
    else vmax = fmax(vmax, cell_inv_dt<NDIM>(U, M.gamma, dx, bad));
  }
  wave_flush(M.scal, vmax, bad);
}

// dt_next = cfl / max_cells(inv dt); advance: t += dt (of the finished step)
__global__ void finalize_kernel(const MeshDev *__restrict__ meshes, int n_meshes, int advance) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n_meshes) return;
  double *sc = meshes[m].scal;
  const double mx = sc[kMaxInv];
  const double next = mx > 0.0 ? meshes[m].cfl * (1.0 / mx) : 0.0;
  if (advance) sc[kTime] += sc[kDt];
  sc[kDt] = next;
  sc[kMaxInv] = 0.0;
}

// Flux fixing (Sec. 2.7) of the coarse blocks with F2C faces.  Each coarse
// face cell is corrected by dt_s (F_c - <F_f>) / dx on a + face,
// dt_s (<F_f> - F_c) / dx on a - face, with <F_f> the FP64 pairwise mean of the
// 2^(d-1) fine fluxes, faces in face order, the state rounded after each.  In
// stage 2 the CFL limit of the corrected cells is then added to the reduction.
//
// One thread per corrected cell, over `parts` workgroups per block: the first
// F2C face of a cell (in face order) names the thread that applies all of its
// corrections, to all variables, and takes its CFL limit.  All faces of a block
// run at once and every load but the flux slots' is independent; face after face
// with a barrier between and the CFL limits in a second pass it was a chain of
// up to a dozen loads.  Launch times, then and now: 264 blocks of 8^3, FP32, 10.3
// and 7.4 us; the 16^3 blocks around a ball refined once in 6^3 trees, FP64, 18.5
// and 11.2 us.
template <typename T, int NDIM, int NV>
__global__ __launch_bounds__(256) void fluxfix_kernel(const MeshDev *__restrict__ Mp, int stage, int parts,
                                                      SubStep ss) {
  const MeshDev &M = *Mp;
  constexpr int NF = 2 * NDIM;
  constexpr int PER = 1 << (NDIM - 1);
  const int32_t cb = M.fix_list[blockIdx.x / parts];
  const int first = (int)(blockIdx.x % parts) * 256 + (int)threadIdx.x, step = parts * 256;
  const int N = M.N, H = N / 2, g = M.g, P = N + 2 * g;
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  const int ob = stage >= 3 ? role_buffer(ss.out, M.cur) : (stage == 1 ? 1 - M.cur : M.cur);
  T *uo = (T *)M.s[ob] + (int64_t)cb * sv * NV;
  const double dx = ldexp(M.dx0, -M.level[cb]);
  const double dts = stage >= 3 ? ss.c * M.scal[kDt] : (stage == 1 ? M.scal[kDt] : 0.5 * M.scal[kDt]);
  const int fv = (NDIM == 3) ? N * N : N;  // face values per variable
  const T *bf = (const T *)M.bflux_f;
  const T *bc = (const T *)M.bflux_c;
  const bool limit = stage == 2 || (stage >= 3 && ss.epi);
  int grp[NF];  // flux slot of each F2C face, -1: no F2C face
#pragma unroll
  for (int f = 0; f < NF; f++) {
    const int info = M.face_info[(int64_t)cb * NF + f];
    grp[f] = (info >= 0 && (info & 1)) ? info >> 1 : -1;
  }
  double vmax = 0.0;
  bool bad = false;
  for (int e = first; e < NF * fv; e += step) {
    const int fe = e / fv, r = e - fe * fv;
    const int p1 = r % N, p2 = r / N, ax = fe >> 1;
    // the face cell's coordinates (tangential axes in increasing order)
    const int in = (fe & 1) ? N - 1 : 0;
    const int c0 = ax == 0 ? in : p1, c1 = ax == 0 ? p1 : ax == 1 ? in : p2, c2 = NDIM == 2 ? 0 : ax == 2 ? in : p2;
    int mine = -1;  // the cell's first F2C face
#pragma unroll
    for (int f = NF - 1; f >= 0; f--) {
      const int c = f < 2 ? c0 : f < 4 ? c1 : c2;
      if (grp[f] >= 0 && c == ((f & 1) ? N - 1 : 0)) mine = f;
    }
    if (mine != fe) continue;
    const int64_t o = cell_off<NDIM>(c0, c1, c2, N, g);
    T u[NV];
#pragma unroll
    for (int v = 0; v < NV; v++) u[v] = uo[v * sv + o];
#pragma unroll
    for (int f = 0; f < NF; f++) {
      const int c = f < 2 ? c0 : f < 4 ? c1 : c2;
      if (grp[f] < 0 || c != ((f & 1) ? N - 1 : 0)) continue;
      const int q1 = f < 2 ? c1 : c0, q2 = NDIM == 2 ? 0 : f < 4 ? c2 : c1;
      const int b1 = q1 >= H, b2 = (NDIM == 3) ? (q2 >= H) : 0;
      const int32_t kf = M.f2c[4 * (grp[f] * PER + b1 + 2 * b2) + 3];
      const int64_t fo = (NDIM == 3 ? (int64_t)(2 * (q2 - b2 * H)) * N : 0) + 2 * (q1 - b1 * H);
#pragma unroll
      for (int v = 0; v < NV; v++) {
        const double Fc = (double)bc[((int64_t)grp[f] * NV + v) * fv + (int64_t)q2 * N + q1];
        const T *ff = bf + ((int64_t)kf * NV + v) * fv + fo;
        double mean;
        if constexpr (NDIM == 3) {
          const double s0 = (double)ff[0] + (double)ff[1];
          const double s1 = (double)ff[N] + (double)ff[N + 1];
          mean = (s0 + s1) * 0.25;
        } else {
          mean = ((double)ff[0] + (double)ff[1]) * 0.5;
        }
        const double corr = (f & 1) ? dts * (Fc - mean) / dx : dts * (mean - Fc) / dx;
        u[v] = (T)((double)u[v] + corr);
      }
    }
#pragma unroll
    for (int v = 0; v < NV; v++) uo[v * sv + o] = u[v];
    if (limit) {
      double U[NV];
#pragma unroll
      for (int v = 0; v < NV; v++) U[v] = (double)u[v];
      if constexpr (NV == 1) vmax = fmax(vmax, inv_dt_adv<NDIM>(M, U[0], dx, bad));
      else vmax = fmax(vmax, cell_inv_dt<NDIM>(U, M.gamma, dx, bad));
    }
  }
  if (limit) wave_flush(M.scal, vmax, bad);
}

// per-block interior sums of every variable in FP64 times the cell volume
template <typename T, int NDIM, int NV>
__global__ __launch_bounds__(256) void totals_kernel(const MeshDev *__restrict__ Mp, double *part) {
  const MeshDev &M = *Mp;
  __shared__ double red[4][NV];
  const int64_t b = blockIdx.x;
  const int N = M.N, g = M.g, P = N + 2 * g;
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  const T *u = (const T *)M.s[M.cur] + b * sv * NV;
  const int cells = (NDIM == 3) ? N * N * N : N * N;
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; v++) acc[v] = 0.0;
  for (int c = threadIdx.x; c < cells; c += blockDim.x) {
    const int i = c % N, j = (c / N) % N, k = (NDIM == 3) ? c / (N * N) : 0;
    const int64_t o = cell_off<NDIM>(i, j, k, N, g);
#pragma unroll
    for (int v = 0; v < NV; v++) acc[v] += (double)u[v * sv + o];
  }
#pragma unroll
  for (int v = 0; v < NV; v++)
    for (int o = 32; o > 0; o >>= 1) acc[v] += __shfl_xor(acc[v], o);
  if ((threadIdx.x & 63) == 0)
    for (int v = 0; v < NV; v++) red[threadIdx.x >> 6][v] = acc[v];
  __syncthreads();
  if (threadIdx.x < NV) {
    const double dx = ldexp(M.dx0, -M.level[b]);
    const double vol = (NDIM == 3) ? dx * dx * dx : dx * dx;
    const int v = threadIdx.x;
    part[b * NV + v] = (((red[0][v] + red[1][v]) + red[2][v]) + red[3][v]) * vol;
  }
}

// fixed-order sum over blocks (one workgroup, deterministic)
__global__ __launch_bounds__(256) void totals_sum_kernel(const double *part, int64_t nb, int nv, double *out) {
  __shared__ double red[256];
  for (int v = 0; v < nv; v++) {
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < nb; b += 256) s += part[b * nv + v];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[v] = red[0];
    __syncthreads();
  }
}

// Instantiation by (element type, dimension, variables): the Euler system
// (ndim + 2 variables) or scalar advection (one).
#define F4_BY_TYPE(KERNEL, GRID, ...)                                                        \
  do {                                                                                       \
    if (nv == 1) {                                                                           \
      if (ndim == 3) {                                                                       \
        if (f64) KERNEL<double, 3, 1><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                   \
        else KERNEL<float, 3, 1><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                        \
      } else {                                                                               \
        if (f64) KERNEL<double, 2, 1><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                   \
        else KERNEL<float, 2, 1><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                        \
      }                                                                                      \
    } else if (ndim == 3) {                                                                  \
      if (f64) KERNEL<double, 3, 5><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                     \
      else KERNEL<float, 3, 5><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                          \
    } else {                                                                                 \
      if (f64) KERNEL<double, 2, 4><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                     \
      else KERNEL<float, 2, 4><<<(GRID), 256, 0, s>>>(__VA_ARGS__);                          \
    }                                                                                        \
  } while (0)

hipError_t launch_dt_full(const foap4_mesh *m, hipStream_t s) {
  if (m->topo.leaves.empty()) return hipSuccess;
  const unsigned nb = (unsigned)m->topo.leaves.size();
  const bool f64 = m->d.prec == FOAP4_F64;
  const int ndim = m->d.ndim, nv = m->nvar;
  F4_BY_TYPE(dt_full_kernel, nb, m->d_dev);
  return hipGetLastError();
}

hipError_t launch_finalize(const MeshDev *d_meshes, int n_meshes, int advance, hipStream_t s) {
  finalize_kernel<<<(n_meshes + 63) / 64, 64, 0, s>>>(d_meshes, n_meshes, advance);
  return hipGetLastError();
}

hipError_t launch_fluxfix(const MeshDev *d_mesh, int ndim, int nv, bool f64, int block_n, int n_fix, int stage,
                          hipStream_t s, const SubStep &ss) {
  if (n_fix <= 0) return hipSuccess;
  // one cell a thread
  const int parts = (2 * ndim * (ndim == 3 ? block_n * block_n : block_n) + 255) / 256;
  F4_BY_TYPE(fluxfix_kernel, n_fix * parts, d_mesh, stage, parts, ss);
  return hipGetLastError();
}

// Fixed device scratch of foap4_conserved_totals_noalloc: the per-block
// partial sums of launch_totals.  One copy per GPU, held until the process
// ends; its address on a device comes from hipGetSymbolAddress with that
// device current (the array's name is not a device address in host code).
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

namespace {
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  double *p = nullptr;
  const hipError_t e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = p;
  return hipSuccess;
}

double *noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

hipError_t launch_totals(const foap4_mesh *m, double *d_part, double *d_out, hipStream_t s) {
  const int64_t nb = (int64_t)m->topo.leaves.size();
  if (nb == 0) return hipSuccess;
  const bool f64 = m->d.prec == FOAP4_F64;
  const int ndim = m->d.ndim, nv = m->nvar;
  F4_BY_TYPE(totals_kernel, (unsigned)nb, m->d_dev, d_part);
  totals_sum_kernel<<<1, 256, 0, s>>>(d_part, nb, m->nvar, d_out);
  return hipGetLastError();
}

#undef F4_BY_TYPE

}  // namespace f4
