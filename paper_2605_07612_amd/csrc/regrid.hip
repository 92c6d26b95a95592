// Refinement flags (Sec. 3.3) and the data remap after a mesh change (Sec. 2.2).
#include "foap4_internal.h"

namespace f4 {

// Lohner-type criterion of eq. lohner-simple on the density, in FP64 with
// the operation order of the definition and no contraction, so that the
// flags equal a plain evaluation bit for bit.  One workgroup per block.
template <typename T, int NDIM, int NV>
__global__ __launch_bounds__(1024) void lohner_kernel(const MeshDev *__restrict__ Mp, double cr2, double cd2,
                                                     double eps, double eps_abs, int8_t *flags,
                                                     const int8_t *skip) {
#pragma clang fp contract(off)
  const MeshDev &M = *Mp;
  const int64_t b = blockIdx.x;
  if (skip && skip[b]) return;
  const int N = M.N, g = M.g, P = N + 2 * g;
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  const T *u = (const T *)M.s[M.cur] + b * sv * NV;  // variable 0 = density
  const int cells = (NDIM == 3) ? N * N * N : N * N;
  bool any_ref = false, all_deref = true;
  for (int c = threadIdx.x; c < cells; c += blockDim.x) {
    const int i = c % N, j = (c / N) % N, k = (NDIM == 3) ? c / (N * N) : 0;
    const double uc = u[cell_off<NDIM>(i, j, k, N, g)];
    double S = 0.0;
#pragma unroll
    for (int d = 0; d < NDIM; d++) {
      const int dm[3] = {d == 0, d == 1, d == 2};
      const double um = u[cell_off<NDIM>(i - dm[0], j - dm[1], k - dm[2], N, g)];
      const double up = u[cell_off<NDIM>(i + dm[0], j + dm[1], k + dm[2], N, g)];
      const double num = fabs((um - 2.0 * uc) + up);
      const double den = ((eps_abs + fabs(uc - um)) + fabs(up - uc)) + eps * ((fabs(um) + 2.0 * fabs(uc)) + fabs(up));
      const double E = num / den;
      S = (d == 0) ? E * E : S + E * E;
    }
    any_ref |= S > cr2;
    all_deref &= S < cd2;
  }
  const int r = __syncthreads_or(any_ref ? 1 : 0);
  const int dall = __syncthreads_and(all_deref ? 1 : 0);
  if (threadIdx.x == 0) flags[b] = r ? 1 : (dall ? -1 : 0);
}

// map[n] = (op, src, arg) of every new block n: op 0 copy old block src, op 1
// prolong child arg (bits x + 2y + 4z) of old block src with limited slopes
// (old ghosts filled), op 2 restrict old children src .. src + 2^d - 1.
//
// A workgroup takes one variable of one new block, or one of `parts` parts of
// it, and each thread moves what lies together: 16 bytes of a copied plane, the
// two fine cells that share a coarse cell along x, the four pairs of fine cells
// under a coarse one.  With one workgroup per block and one value per thread and
// round (80 rounds of a load each for an FP64 16^3 block) it was bound by load
// latency: 216 FP64 16^3 blocks, a ball of them refined and coarsened again: 114
// us a launch, 30 us now.
template <typename T, int NDIM, int NV, int N>
__device__ __forceinline__ void remap_block(const T *__restrict__ uold, T *unew, int op, int64_t src, int arg,
                                            int64_t n, int v, int g, int first, int step) {
  // FP64 in the operation order of the definitions, no contraction (the
  // prolonged value u_P + corr / 4 stays bit-exact when corr / 4 is subnormal)
#pragma clang fp contract(off)
  typedef T Pair __attribute__((ext_vector_type(2)));
  constexpr int H = N / 2, CELLS = NDIM == 3 ? N * N * N : N * N;
  const int P = N + 2 * g;
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  const int64_t bel = sv * NV;
  auto at = [&](int i, int j, int k) -> int { return cell_off<NDIM>(i, j, k, N, g); };
  T *un = unew + n * bel + v * sv;
  if (op == 0) {
    // an interior plane is N^2 contiguous values, and every offset is a
    // multiple of 16 bytes: N is a multiple of 8, P and so the strides of a
    // variable and a block are even (2D: P^2 a multiple of 4)
    constexpr int W = 16 / (int)sizeof(T);
    typedef T Vec __attribute__((ext_vector_type(W)));
    const T *uo = uold + src * bel + v * sv;
    constexpr int B = 4;  // loads in flight per thread
    for (int e0 = first; e0 < CELLS / W; e0 += B * step) {
      Vec val[B];
#pragma unroll
      for (int q = 0; q < B; q++) {
        const int c = (e0 + q * step) * W;
        if (c < CELLS) val[q] = *(const Vec *)(uo + at(0, 0, c / (N * N)) + c % (N * N));
      }
#pragma unroll
      for (int q = 0; q < B; q++) {
        const int c = (e0 + q * step) * W;
        if (c < CELLS) *(Vec *)(un + at(0, 0, c / (N * N)) + c % (N * N)) = val[q];
      }
    }
  } else if (op == 1) {
    const T *uc = uold + src * bel + v * sv;
    for (int e = first; e < CELLS / 2; e += step) {
      const int hi = e % H, j = (e / H) % N, k = NDIM == 3 ? e / (H * N) : 0;
      const int pc[3] = {(arg & 1) * H + hi, ((arg >> 1) & 1) * H + (j >> 1),
                         NDIM == 3 ? ((arg >> 2) & 1) * H + (k >> 1) : 0};
      const double up = uc[at(pc[0], pc[1], pc[2])];
      double delta[NDIM];
#pragma unroll
      for (int d = 0; d < NDIM; d++) {
        const int dx = d == 0, dy = d == 1, dz = d == 2;
        const double a = up - (double)uc[at(pc[0] - dx, pc[1] - dy, pc[2] - dz)];
        const double bb = (double)uc[at(pc[0] + dx, pc[1] + dy, pc[2] + dz)] - up;
        delta[d] = 0.0;
        if (a > 0.0 && bb > 0.0) delta[d] = a < bb ? a : bb;
        else if (a < 0.0 && bb < 0.0) delta[d] = a > bb ? a : bb;
      }
      Pair out;
#pragma unroll
      for (int s = 0; s < 2; s++) {
        double corr = s ? delta[0] : -delta[0];
        corr = corr + ((j & 1) ? delta[1] : -delta[1]);
        if constexpr (NDIM == 3) corr = corr + ((k & 1) ? delta[2] : -delta[2]);
        out[s] = (T)(up + 0.25 * corr);
      }
      *(Pair *)(un + at(2 * hi, j, k)) = out;
    }
  } else {
    for (int e = first; e < CELLS; e += step) {
      const int i = e % N, j = (e / N) % N, k = NDIM == 3 ? e / (N * N) : 0;
      const int bx = i >= H, by = j >= H, bz = NDIM == 3 ? k >= H : 0;
      const int x = 2 * (i - bx * H), y = 2 * (j - by * H), z = NDIM == 3 ? 2 * (k - bz * H) : 0;
      const T *uq = uold + (src + (bx + 2 * by + 4 * bz)) * bel + v * sv;
      auto pair = [&](int yy, int zz) -> Pair { return *(const Pair *)(uq + at(x, yy, zz)); };
      double val;
      if constexpr (NDIM == 2) {
        const Pair f0 = pair(y, 0), f1 = pair(y + 1, 0);
        val = (((double)f0[0] + (double)f0[1]) + ((double)f1[0] + (double)f1[1])) * 0.25;
      } else {
        const Pair f0 = pair(y, z), f1 = pair(y + 1, z), f2 = pair(y, z + 1), f3 = pair(y + 1, z + 1);
        const double a0 = (double)f0[0] + (double)f0[1], a1 = (double)f1[0] + (double)f1[1];
        const double a2 = (double)f2[0] + (double)f2[1], a3 = (double)f3[0] + (double)f3[1];
        val = ((a0 + a1) + (a2 + a3)) * 0.125;
      }
      un[at(i, j, k)] = (T)val;
    }
  }
}

template <typename T, int NDIM, int NV>
__global__ __launch_bounds__(256) void remap_kernel(const T *__restrict__ uold, T *unew, const int32_t *map, int N,
                                                    int g, int parts) {
  const int64_t item = blockIdx.x / parts, n = item / NV;
  const int v = (int)(item % NV), first = (int)(blockIdx.x % parts) * 256 + (int)threadIdx.x, step = parts * 256;
  const int op = map[3 * n], src = map[3 * n + 1], arg = map[3 * n + 2];
  switch (N) {
    case 8: remap_block<T, NDIM, NV, 8>(uold, unew, op, src, arg, n, v, g, first, step); break;
    case 16: remap_block<T, NDIM, NV, 16>(uold, unew, op, src, arg, n, v, g, first, step); break;
    default: remap_block<T, NDIM, NV, 32>(uold, unew, op, src, arg, n, v, g, first, step); break;
  }
}

// Instantiation by (element type, dimension, variables): the Euler system
// (ndim + 2 variables) or scalar advection (one).
#define F4_BY_TYPE(KERNEL, T_, GRID, THREADS, ...)                                                 \
  do {                                                                                    \
    if (f64) {                                                                            \
      using T_ = double;                                                                  \
      if (nv == 1) {                                                                      \
        if (ndim == 3) KERNEL<T_, 3, 1><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);              \
        else KERNEL<T_, 2, 1><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);                        \
      } else if (ndim == 3) KERNEL<T_, 3, 5><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);         \
      else KERNEL<T_, 2, 4><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);                          \
    } else {                                                                              \
      using T_ = float;                                                                   \
      if (nv == 1) {                                                                      \
        if (ndim == 3) KERNEL<T_, 3, 1><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);              \
        else KERNEL<T_, 2, 1><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);                        \
      } else if (ndim == 3) KERNEL<T_, 3, 5><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);         \
      else KERNEL<T_, 2, 4><<<(GRID), (THREADS), 0, s>>>(__VA_ARGS__);                          \
    }                                                                                     \
  } while (0)

hipError_t launch_lohner(const foap4_mesh *m, int8_t *d_flags, const int8_t *skip, hipStream_t s) {
  const int64_t nb = (int64_t)m->topo.leaves.size();
  if (nb == 0) return hipSuccess;
  const double cr = 5e-2, cd = 6.25e-3;  // c_refine, c_derefine of the AMR runs (Sec. 5.4)
  const double cr2 = cr * cr, cd2 = cd * cd, eps = 1e-2, eps_abs = 1e-10;
  const bool f64 = m->d.prec == FOAP4_F64;
  const int ndim = m->d.ndim, nv = m->nvar;
  // at most four cells a thread but for 32^3 blocks: each round is a load's latency
  const int cells = ndim == 3 ? m->d.block_n * m->d.block_n * m->d.block_n : m->d.block_n * m->d.block_n;
  const int threads = cells > 1024 ? 1024 : 256;
  F4_BY_TYPE(lohner_kernel, T, (unsigned)nb, threads, m->d_dev, cr2, cd2, eps, eps_abs, d_flags, skip);
  return hipGetLastError();
}

hipError_t launch_remap(const foap4_mesh *m, const void *src_state, void *dst_state, const int32_t *d_map,
                        int64_t nb_new, hipStream_t s) {
  if (nb_new == 0) return hipSuccess;
  const bool f64 = m->d.prec == FOAP4_F64;
  const int N = m->d.block_n, g = m->d.n_ghost;
  const int ndim = m->d.ndim, nv = m->nvar;
  const int parts = (ndim == 3 ? N * N * N : N * N) > 2048 ? (N == 32 ? 16 : 2) : 1;  // at most 8 cells a thread
  F4_BY_TYPE(remap_kernel, T, (unsigned)(nb_new * nv * parts), 256, (const T *)src_state, (T *)dst_state, d_map, N, g,
             parts);
  return hipGetLastError();
}

#undef F4_BY_TYPE

}  // namespace f4
